// 16-bit MFMA kernels for gfx950 used when many tokens go through the layers at once (prefill and
// scoring): weight packing, the token-parallel ("big") GEMM, and the fused LM head of the scoring
// pass (log-softmax + target gather).
//
// Operand type: the model's weights are bf16 values; the packed copies hold the same values as IEEE
// half (exact for 6.1e-5 <= |w| <= 65504, absolute error below 3e-8 under that) and activations
// are rounded to half (clamped to its range) instead of bf16.  Both run the MFMA at the same rate;
// half keeps 3 more mantissa bits, which is what keeps 28-layer models inside the stated logit and
// log-prob tolerances (with bf16 activations the rounding points alone put the 1.5B-class model's
// logits 6e-2 away from the definition).
#include "tiles.h"
#include "ranges.h"
#include <algorithm>
#include <type_traits>

namespace sapo {

// ---------------------------------------------------------------------------------------
// Filling a handle: every matrix, row-major bf16 [n_rows, K], goes out as half in both fragment orders (W32 and W16), every
// gain is copied, in a few launches for the whole model: a launch per tensor and order was 400 launches of a few us each with
// as much between them (0.5B: 5.2 ms, of which the kernels 1.6; now 1.1).
// A wave takes 32 rows x 64 k: every value is read once (8 rows x 128 contiguous bytes per request) and stored as the same 16
// bytes in either order, 128 contiguous bytes per eight rows.
// half 0, 1 instead of -1 (gate, up): 16 rows go into rows 16 half .. 16 half + 15 of each 32-row tile, so that an accumulator
// block of 32 features holds 16 gate features and, two register quads on in the same lane, the up features that belong to
// them: a kernel may take any number of blocks.  16-row tile t goes to tile16 + t stride16.
// range: kPackRangeSlots (512) pairs of counters, to be summed by the reader.  The first of a pair counts values half
// cannot hold (|w| > 65504, infinities, NaN: they would be clamped or carried as NaN), the second non-zero values
// below half's smallest normal number 2^-14 (kept with an absolute error below 3e-8).
// ---------------------------------------------------------------------------------------
constexpr int kPackTasks = 48;   // tasks of a launch: they travel as kernel arguments (at most 4 KiB)
struct PackTasks { int n; PackTask t[kPackTasks]; };
static_assert(sizeof(PackTasks) + 64 <= 4096, "kernel arguments");

__global__ void __launch_bounds__(256) k_pack_weights(PackTasks tasks, unsigned* __restrict__ range) {
  int ti = 0;
  for (int end = tasks.n; end - ti > 1;) {
    const int mid = (ti + end) >> 1;
    if ((int)blockIdx.x >= tasks.t[mid].first_block) ti = mid; else end = mid;
  }
  const PackTask t = tasks.t[ti];
  const int lane = threadIdx.x & 63, block = (int)blockIdx.x - t.first_block;
  if (t.dst32 == nullptr) {   // a gain: n_rows floats
    for (int i = threadIdx.x; i < t.n_rows; i += 256) ((float*)t.dst16)[i] = ((const float*)t.src)[i];
    return;
  }
  const int units_k = t.K >> 6, unit = block * 4 + wave_index(threadIdx.x);
  if (unit >= (t.n_rows >> 5) * units_k) return;   // a wave leaves as a whole
  const int r32 = unit / units_k, k0 = (unit - r32 * units_k) * 64, k8 = lane & 7;
  Frag v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i].u = *(const uint4*)((const bf16*)t.src + (size_t)(r32 * 32 + 8 * i + (lane >> 3)) * t.K + k0 + k8 * 8);
  unsigned too_large = 0, tiny = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = r32 * 32 + 8 * i + (lane >> 3);
    Frag o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float w = (float)v[i].v[e], a = fabsf(w);   // bf16 value -> half
      o.h[e] = from_f32<f16>(w);
      too_large += !(a <= 65504.f);
      tiny += (a > 0.f && a < 6.103515625e-05f);
    }
    const size_t ks = (k0 >> 4) + (k8 >> 1);
    const int tile = t.half < 0 ? row >> 5 : row >> 4, in = t.half < 0 ? row & 31 : t.half * 16 + (row & 15);
    t.dst32[((size_t)(t.tile32 + tile) * (t.K >> 4) + ks) * 64 + (k8 & 1) * 32 + in] = o.u;
    t.dst16[((size_t)(t.tile16 + (row >> 4) * t.stride16) * (t.K >> 5) + (k0 >> 5) + (k8 >> 2)) * 64 + (k8 & 3) * 16 + (row & 15)] = o.u;
  }
  // one atomic per wave and counter, only when there is something to add, spread over kPackRangeSlots pairs of
  // counters (small weights are common: with one pair every wave of a 0.5B model queues on the same address)
  unsigned packed = (too_large << 16) | tiny;          // at most 32 each per lane, 2048 each per wave
  for (int off = 32; off > 0; off >>= 1) packed += __shfl_xor(packed, off, 64);
  if (lane == 0) {
    unsigned* slot = range + 2 * (((unsigned)(unit + blockIdx.x) * 2654435761u) >> (32 - 9));
    if (packed >> 16) atomicAdd(slot, packed >> 16);
    if (packed & 0xffffu) atomicAdd(slot + 1, packed & 0xffffu);
  }
}
hipError_t m_pack_weights(const PackTask* tasks, int n, unsigned* range, hipStream_t st) {
  for (int i = 0; i < n; ++i)
    if (tasks[i].dst32 && (tasks[i].n_rows % 32 != 0 || tasks[i].K % 64 != 0)) return hipErrorInvalidValue;
  for (int i0 = 0; i0 < n; i0 += kPackTasks) {
    PackTasks a;
    a.n = n - i0 < kPackTasks ? n - i0 : kPackTasks;
    int blocks = 0;
    for (int i = 0; i < a.n; ++i) {
      a.t[i] = tasks[i0 + i];
      a.t[i].first_block = blocks;
      blocks += a.t[i].dst32 ? (a.t[i].n_rows / 32 * (a.t[i].K / 64) + 3) / 4 : 1;
    }
    const hipError_t e = launch(KID_MISC, k_pack_weights, dim3(blocks), dim3(256), 0, st, a, range);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// =======================================================================================
// Token-parallel ("big") GEMM:  C[tok, feat] = sum_k X[tok, k] W[feat, k]
//
// Both operands are in 32-row fragment order in global memory (one MFMA 32x32x16 operand of one
// wave = one contiguous 1 KiB block):
//   W32[((fblk * KS + ks) * 64 + lane)] = W[fblk*32 + lane%32][ks*16 + (lane/32)*8 .. +7],  KS = K / 16
//   X32[((tblk * KS + ks) * 64 + lane)] = X[tblk*32 + lane%32][ks*16 + (lane/32)*8 .. +7]
// Workgroup tile 128 TJ tokens x 128 features, 4 waves, each 32 TJ tokens x all 128 features = 4 x TJ MFMA tiles; H
// 16-k steps per stage.  The token operand goes from global memory straight into the registers of the one wave that
// uses it, two stages ahead; the feature operand, which all four waves read, goes through a three-stage LDS ring filled by
// direct-to-LDS copies.  What bounds the loop is the LDS: with both operands in the ring and waves of 128 tokens x
// 64 features (what this replaces) a wave read 0.75 KB and the copies wrote 0.375 KB of LDS per MFMA, more than a compute
// unit's LDS delivers in the MFMA's time; now it is 0.5 + 0.125 KB.  Stand-alone, random operands (old -> H = 2 -> H = 4):
// 49152 x 9728 x 896 870 -> 770 -> 697 us, 49152 x 896 x 4864 401 -> 387 -> 368 us, 49152 x 17920 x 1536 2350 -> 2170 ->
// 2125 us (1.27 PFLOP/s; the rest is the clock that the matrix cores hold under this load).
// TJ = 2: two workgroups per compute unit (48 KiB LDS, <= 256 registers), which is what overlaps one workgroup's barrier
// and LDS latency with the other's MFMAs; TJ = 1: three.
// All requests of the loop are issued from inline assembly and awaited with explicit s_waitcnt vmcnt(N) (they retire in
// order): the compiler would wait for the copies before any LDS read, and for the newest request before the oldest
// register's use.
// Accumulator layout: acc[fi][tj][4 r + j] = C[tok = wave * 32 TJ + tj*32 + lane%32][feat = fi*32 + 8 r + (lane/32)*4 + j].
// ---------------------------------------------------------------------------------------
constexpr int kRing = 3;                                            // stages of the LDS ring
constexpr int ring_bytes(int H) { return kRing * 4 * H * 1024; }     // 4 H fragments of 1 KiB per stage
constexpr int kBigLds = ring_bytes(4);

// Rows of a launch for at most M (PK: as many as `rows`, on the device, says).  A template parameter of the kernels, because what
// they execute before their first requests counts: with a test of the pointer a scoring call of 301 tokens took 1.465 ms instead of 1.444.
// Through the vector path: a scalar load, the same for every lane, would be waited for with all other scalar loads on their way,
// and those of the arguments that are not preloaded take longer.  16 x 256 tokens, 1.5B, us without a row count, with it as a
// scalar load, and like this: down 131.1, 135.2, 131.8; gate/up 200.2, 201.5, 200.4; the scoring call 12570, 12677, 12525.
template <bool PK> __device__ __forceinline__ int rows_there(const int* rows, int M) {
  if constexpr (PK) return min(M, __builtin_amdgcn_readfirstlane(__hip_atomic_load(rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)));
  return M;
}
__device__ __forceinline__ bool big_raster(int NX, int NY, int& bx, int& by) {
  const bool any = tile_of_block(blockIdx.x, NX, NY, bx, by);
  bx = __builtin_amdgcn_readfirstlane(bx);   // the quotients come out of vector registers: addresses would stay there
  by = __builtin_amdgcn_readfirstlane(by);
  return any;
}
static int big_grid(int NX, int NY) { return tile_blocks(NX, NY); }

// The k loop of one tile.  begin() requests the first two stages, run() multiplies all of them; a caller that walks several
// tiles may call begin() for the next one before it is done with the accumulators, after a barrier (the ring is free
// once every wave has left run()).
template <int TJ, int H>
struct TileLoop {
  static constexpr int NF = H;                // ring copies per wave and stage: the H fragments of a feature block
  static_assert(H == 2 || H == 4, "stage of 32 or 64 k");
  u32x4 x[2][H][TJ];
  const char* wbase;          // this wave's fragments of the feature operand
  const char* xbase[TJ];
  const char* xrow;           // start of the token operand
  unsigned off, ring;         // lane offset; LDS address of this wave's fragments in the ring's stage 0
  int nst;

  // X rows tblk0 * 32 .. (token blocks past the last one, n_tblk - 1, repeat it: their results are never stored), W rows
  // fblk0 * 32 .. + 127, n_stages stages of 16 H k from 16-k step ks0 on
  __device__ __forceinline__ void tokens(const uint4* Xp, int n_tblk, int KS, int tblk0, int ks0) {
    const int wave = wave_index(threadIdx.x);
#pragma unroll
    for (int t = 0; t < TJ; ++t) {
      const int tb = min(tblk0 + wave * TJ + t, n_tblk - 1);
      xbase[t] = (const char*)(Xp + ((size_t)tb * KS + ks0) * 64);
    }
  }
  // ring fragment f of a stage: feature block f / H, 16-k step f % H; wave w copies those of block w
  __device__ __forceinline__ void features(const uint4* Wp, int KS, int fblk0, int ks0, int n_stages, const uint4* smem) {
    const int wave = wave_index(threadIdx.x);
    wbase = (const char*)(Wp + ((size_t)(fblk0 + wave) * KS + ks0) * 64);
    ring = __builtin_amdgcn_readfirstlane(lds_addr(smem)) + (unsigned)(wave * NF * 1024);
    off = (threadIdx.x & 63) * 16;
    nst = n_stages;
  }
  template <int I> __device__ __forceinline__ void request_w(int st) {
    dma16(wbase + (size_t)st * (H * 1024) + I * 1024, off, ring + (unsigned)((st % kRing) * (4 * H * 1024) + I * 1024));
  }
  __device__ __forceinline__ void request_ws(int st) {
    request_w<0>(st);
    if constexpr (NF >= 2) request_w<1>(st);
    if constexpr (NF == 4) { request_w<2>(st); request_w<3>(st); }
  }
  template <int HH> __device__ __forceinline__ void request_x(int p, int st) {
#pragma unroll
    for (int t = 0; t < TJ; ++t) reg16<HH * 1024>(x[p][HH][t], xbase[t] + (size_t)st * (H * 1024), off);
  }
  // LIVE = false: a wave all of whose tokens lie past the end copies its feature blocks and multiplies nothing
  template <bool LIVE = true> __device__ __forceinline__ void begin() {
    auto stage = [&](auto pc) {
      constexpr int p = decltype(pc)::value;
      request_ws(p);
      if constexpr (LIVE) {
        request_x<0>(p, p); request_x<1>(p, p);
        if constexpr (H == 4) { request_x<2>(p, p); request_x<3>(p, p); }
      }
    };
    stage(std::integral_constant<int, 0>());
    if (nst > 1) stage(std::integral_constant<int, 1>());
  }
  template <int P, bool LIVE> __device__ __forceinline__ void stage(int st, const uint4* smem, f32x16 (&acc)[4][TJ]) {
    constexpr int PER = NF + (LIVE ? TJ * H : 0);   // requests per wave and stage
    // this wave's requests of stage st have landed once at most the next stage's are outstanding ...
    if (st + 1 < nst) wait_vmcnt<PER>(); else wait_vmcnt<0>();
    if constexpr (LIVE) {
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int t = 0; t < TJ; ++t) landed(x[P][h][t]);
    }
    wg_barrier();   // ... and everybody's; stage st - 1 is consumed
    const bool more = st + 2 < nst;
    if constexpr (!LIVE) {
      if (more) request_ws(st + 2);
    } else {
      const uint4* buf = smem + (st % kRing) * (4 * H * 64) + (threadIdx.x & 63);
      auto step = [&](auto hc) {
        constexpr int h = decltype(hc)::value;
        Frag w[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) w[f].u = buf[(f * H + h) * 64];
        __builtin_amdgcn_s_setprio(1);
        // The ring copies of stage st + 2 go out one after each of the first MFMAs, a step's registers are requested again
        // right after their last use; the fences keep the compiler from regrouping them.
        auto feature = [&](auto fc) {
          constexpr int f = decltype(fc)::value;
#pragma unroll
          for (int t = 0; t < TJ; ++t) {
            Frag xx; xx.n = x[P][h][t];
            acc[f][t] = mfma32(w[f], xx, acc[f][t]);
          }
          if constexpr (h * 4 + f < NF) {
            __builtin_amdgcn_sched_barrier(0);
            if (more) request_w<h * 4 + f>(st + 2);
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        feature(std::integral_constant<int, 0>()); feature(std::integral_constant<int, 1>());
        feature(std::integral_constant<int, 2>()); feature(std::integral_constant<int, 3>());
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        if (more) request_x<h>(P, st + 2);
        __builtin_amdgcn_sched_barrier(0);
      };
      step(std::integral_constant<int, 0>()); step(std::integral_constant<int, 1>());
      if constexpr (H == 4) { step(std::integral_constant<int, 2>()); step(std::integral_constant<int, 3>()); }
    }
  }
  template <bool LIVE = true> __device__ __forceinline__ void run(const uint4* smem, f32x16 (&acc)[4][TJ]) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    int st = 0;
    for (; st + 1 < nst; st += 2) {
      stage<0, LIVE>(st, smem, acc);
      stage<1, LIVE>(st + 1, smem, acc);
    }
    if (st < nst) stage<0, LIVE>(st, smem, acc);
  }
};

// 1 / rms of the wave's tokens of a tile from the parts of their sums of squares (at most 16 parts, row stride a multiple
// of 4; halves: each part as two): requested behind the first stages, so that they ride on the same latency
template <int TJ>
__device__ __forceinline__ void row_scales(const float* __restrict__ ssq, int parts, bool halves, float norm_dim, float eps, int tok0,
                                           int M, float (&scale)[TJ]) {
  if (halves) {
    const int ps = (2 * parts + 3) & ~3;
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj) {
      const int tok = min(tok0 + tj * 32, M - 1);
      float4 half[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        half[i] = (4 * i < ps) ? *(const float4*)(ssq + (size_t)tok * ps + 4 * i) : make_float4(0.f, 0.f, 0.f, 0.f);
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        ss += (2 * i + 0 < parts) ? half[i].x + half[i].y : 0.f;
        ss += (2 * i + 1 < parts) ? half[i].z + half[i].w : 0.f;
      }
      scale[tj] = rsqrtf(ss / norm_dim + eps);
    }
    return;
  }
  const int ps = (parts + 3) & ~3;
  float4 part[TJ][4];
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) {
    const int tok = min(tok0 + tj * 32, M - 1);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      part[tj][i] = (4 * i < ps) ? *(const float4*)(ssq + (size_t)tok * ps + 4 * i) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // padding slots are never written: select, do not add
      ss += (4 * i + 0 < parts) ? part[tj][i].x : 0.f;
      ss += (4 * i + 1 < parts) ? part[tj][i].y : 0.f;
      ss += (4 * i + 2 < parts) ? part[tj][i].z : 0.f;
      ss += (4 * i + 3 < parts) ? part[tj][i].w : 0.f;
    }
    scale[tj] = rsqrtf(ss / norm_dim + eps);
  }
}

// MODE: the epilogue (BigEpi::mode), each with a register allocation of its own
template <int TJ, int H, int MODE, bool PK>
__global__ void __launch_bounds__(256, TJ == 2 ? 2 : 3) k_gemm_big(const uint4* __restrict__ Xp,
                                                                      const uint4* __restrict__ Wp, const int* rows, int M, int N, int K,
                                                                      BigEpi ep) {
  constexpr int TM = 128 * TJ;   // tokens per tile
  extern __shared__ uint4 smem[];
  int bx, by;
  M = rows_there<PK>(rows, M);
  if (!big_raster(N >> 7, (M + TM - 1) / TM, bx, by)) return;
  f32x16 acc[4][TJ];
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const int tok0 = by * TM + wave * (32 * TJ) + (lane & 31);
  float row_scale[TJ];
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) row_scale[tj] = 1.f;
  {
    TileLoop<TJ, H> loop;
    loop.tokens(Xp, (M + 31) >> 5, K >> 4, by * (4 * TJ), 0);
    loop.features(Wp, K >> 4, bx * 4, 0, K / (16 * H), smem);
    loop.begin();
    if (MODE != BIG_ADD_F32 && ep.ssq_in) row_scales<TJ>(ep.ssq_in, ep.ssq_parts, ep.ssq_halves, ep.norm_dim, ep.eps, tok0, M, row_scale);
    loop.run(smem, acc);
  }
  const int fcol = bx * 128 + (lane >> 5) * 4;   // + fi * 32 + 8 r: this lane's four features of block (fi, r)
  if (MODE != BIG_ADD_F32 && ep.ssq_in) {
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
      for (int fi = 0; fi < 4; ++fi)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[fi][tj][v] *= row_scale[tj];
  }
  if constexpr (MODE == BIG_SWIGLU) {
    const int F = N >> 1;
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj) {
      const int tok = tok0 + tj * 32;
      if (tok >= M) continue;   // lanes l and l + 32 hold the same token: they leave together
#pragma unroll
      for (int fi = 0; fi < 4; ++fi) {
        // a block is 16 gate rows and the 16 matching up rows; act goes out in X32 order over F = N / 2
        const int f0 = (bx * 4 + fi) * 16 + (lane >> 5) * 4;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          f16x4 o;
#pragma unroll
          for (int j = 0; j < 4; ++j) o[j] = from_f32<f16>(silu_f(acc[fi][tj][4 * r + j]) * acc[fi][tj][4 * (r + 2) + j]);
          *(f16x4*)(ep.out_act + x32_chunk(tok, f0 + 8 * r, F >> 4) * 8 + ((lane >> 5) << 2)) = o;
        }
      }
    }
  } else if constexpr (MODE == BIG_STORE_F32) {
#pragma unroll
    for (int fi = 0; fi < 4; ++fi) {
      float4 bb[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        bb[r] = ep.bias ? *(const float4*)(ep.bias + fcol + fi * 32 + 8 * r) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int tj = 0; tj < TJ; ++tj) {
        const int tok = tok0 + tj * 32;
        if (tok >= M) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float4 v = make_float4(acc[fi][tj][4 * r], acc[fi][tj][4 * r + 1], acc[fi][tj][4 * r + 2], acc[fi][tj][4 * r + 3]);
          if (ep.bias) { v.x += bb[r].x; v.y += bb[r].y; v.z += bb[r].z; v.w += bb[r].w; }
          *(float4*)(ep.out_f32 + (size_t)tok * ep.ldc + fcol + fi * 32 + 8 * r) = v;
        }
      }
    }
  }
  if constexpr (MODE == BIG_ADD_F32) {
    // Residual update.  In the accumulator layout a lane holds one token, so a load or store instruction on the
    // row-major fp32 residual touches 32 cache lines for 1 KiB.  The residual therefore moves in row layout (16 lanes
    // cover 256 contiguous bytes of a row: 8 full lines per instruction) and changes layout through LDS, once on the
    // way in and once on the way out, 32 tokens x 64 features at a time in the wave's own part of the ring (rows padded
    // to 68 floats).  The sums, the next operand and the sums of squares are taken in the accumulator layout.  The next
    // pass's rows are requested before a pass's stores go out, since a load issued behind a store also waits for the
    // store's acknowledgement.  A tile without rows past the end and the producer side are compile-time cases, so that
    // the common one is straight-line code whose waits the compiler can count exactly.
    constexpr int RS = 68, NP = 2 * TJ;   // passes: token block tj, feature half fh
    wg_barrier();   // every wave has read its last stage: the ring is free
    float* R = (float*)smem + wave * (32 * RS);
    const int rt = lane >> 4, rc = (lane & 15) * 4;   // row layout: token 4 i + rt of the block, features rc .. rc + 3
    const int row0 = by * TM + wave * (32 * TJ);
    auto wave_sync = [] {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    float ssq_half[TJ][2];
    auto update = [&](auto full_c, auto prod_c) {
      constexpr bool full = decltype(full_c)::value, prod = decltype(prod_c)::value;
      // the tile's 128 gains wait in LDS behind the four row areas (in registers they would not fit next to the rows)
      float* G = (float*)smem + 4 * 32 * RS + wave * 128;
      if (prod && lane < 32) *(float4*)(G + 4 * lane) = *(const float4*)(ep.gain_next + bx * 128 + 4 * lane);
      f32x4 in[8];   // (as HIP's float4, a struct, the array may end up in scratch memory: O 129 -> 175 us)
      auto request = [&](int p) {   // pass p: token block p / 2, feature half p % 2
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int tok = row0 + (p >> 1) * 32 + 4 * i + rt;
          in[i] = (full || tok < M) ? *(const f32x4*)(ep.out_f32 + (size_t)tok * ep.ldc + bx * 128 + (p & 1) * 64 + rc)
                                    : f32x4{0.f, 0.f, 0.f, 0.f};
        }
      };
      request(0);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int tj = p >> 1, fh = p & 1, tok = tok0 + tj * 32;
#pragma unroll
        for (int i = 0; i < 8; ++i) *(f32x4*)(R + (4 * i + rt) * RS + rc) = in[i];
        wave_sync();
        float ssq = 0.f;
#pragma unroll
        for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int fi = 2 * fh + f2;
            float4* q = (float4*)(R + (lane & 31) * RS + f2 * 32 + 8 * r + (lane >> 5) * 4);
            const float4 w = *q;
            const float4 v = make_float4(acc[fi][tj][4 * r] + w.x, acc[fi][tj][4 * r + 1] + w.y,
                                         acc[fi][tj][4 * r + 2] + w.z, acc[fi][tj][4 * r + 3] + w.w);
            *q = v;
            if (prod && (full || tok < M)) {
              ssq += sum_squares4(v);
              const float4 gn = *(const float4*)(G + fi * 32 + 8 * r + (lane >> 5) * 4);
              f16x4 hv;
              hv[0] = from_f32<f16>(v.x * gn.x); hv[1] = from_f32<f16>(v.y * gn.y);
              hv[2] = from_f32<f16>(v.z * gn.z); hv[3] = from_f32<f16>(v.w * gn.w);
              *(f16x4*)(ep.xn_out + x32_chunk(tok, fcol + fi * 32 + 8 * r, N >> 4) * 8 + ((lane >> 5) << 2)) = hv;
            }
          }
        ssq_half[tj][fh] = ssq + __shfl_xor(ssq, 32, 64);
        wave_sync();
        f32x4 out[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = *(const f32x4*)(R + (4 * i + rt) * RS + rc);
        if (p + 1 < NP) request(p + 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int t = row0 + tj * 32 + 4 * i + rt;
          if (full || t < M) *(f32x4*)(ep.out_f32 + (size_t)t * ep.ldc + bx * 128 + fh * 64 + rc) = out[i];
        }
        wave_sync();   // the rows are in registers before the next pass overwrites them
      }
    };
    const bool full = by * TM + TM <= M;
    if (ep.gain_next) {
      if (full) update(std::true_type(), std::true_type());
      else update(std::false_type(), std::true_type());
      if (lane < 32) {
        const int ps = ((N >> 7) + 3) & ~3;
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj)
          if (tok0 + tj * 32 < M) ep.ssq_out[(size_t)(tok0 + tj * 32) * ps + bx] = ssq_half[tj][0] + ssq_half[tj][1];
      }
    } else {
      if (full) update(std::true_type(), std::false_type());
      else update(std::false_type(), std::false_type());
    }
  }
}
// ---------------------------------------------------------------------------------------
// Few tokens (prompts of a few hundred tokens, small scoring calls): the tiles above leave most of the chip idle (at 128
// tokens the 0.5B down projection was 7 workgroups of 2.5 MB, 44 us whatever the number of tokens), and every output's
// sum has to stay one chain of MFMAs over K.  Here a wave owns 32 tokens x NB 32-feature blocks, a workgroup WM x WN such
// waves, and all four waves fetch: both operands go through an LDS ring of D stages of 64 k, 60 .. 144 KiB of requests in
// flight.  Wave w fetches k step w of every stage.  Sums, epilogues and bits are those of the kernels above.  0.5B, one
// sequence of 128 tokens: down 46 -> 24 us, O 13 -> 8, QKV 19 -> 8, gate/up 17 -> 11 (a scoring call 2.64 -> 1.53 ms); 1024
// tokens 3.77 -> 2.95 ms.  What is left is the chain itself: 0.22 us per stage of 64 k (wait, barrier, LDS, MFMAs).
// ---------------------------------------------------------------------------------------
template <int WM, int WN, int NB, int D>
struct MidLoop {
  static constexpr int FX = WM, F = WM + WN * NB;   // token blocks, and fragments of a k step = requests per wave and stage
  static_assert(WM * WN <= 4 && F * (D - 2) <= 63, "four waves; the counter of outstanding requests");
  static constexpr int kBytes = D * 4 * F * 1024;
  const char* base[F];
  unsigned off, ring;
  int nst;
  __device__ __forceinline__ void begin(const uint4* Xp, const uint4* Wp, int n_tblk, int KS, int tblk0, int fblk0, const uint4* smem) {
    const int wave = wave_index(threadIdx.x);
#pragma unroll
    for (int f = 0; f < F; ++f)
      base[f] = (const char*)(f < FX ? Xp + ((size_t)min(tblk0 + f, n_tblk - 1) * KS + wave) * 64
                                     : Wp + ((size_t)(fblk0 + f - FX) * KS + wave) * 64);
    off = (threadIdx.x & 63) * 16;
    ring = __builtin_amdgcn_readfirstlane(lds_addr(smem)) + (unsigned)(wave * F * 1024);
    nst = KS >> 2;
#pragma unroll
    for (int p = 0; p < D - 1; ++p)
      if (p < nst) request(p);
  }
  __device__ __forceinline__ void request(int st) {
    const unsigned dst = ring + (unsigned)((st % D) * (4 * F * 1024));
#pragma unroll
    for (int f = 0; f < F; ++f) dma16(base[f] + (size_t)st * 4096, off, dst + f * 1024u);
  }
  __device__ __forceinline__ void arrive(int st) {
    if (st + D - 2 < nst) wait_vmcnt<F * (D - 2)>(); else wait_vmcnt<0>();   // this wave's part of stage st has landed ...
    wg_barrier();                                                           // ... everybody's has; stage st - 1 is consumed
    if (st + D - 1 < nst) request(st + D - 1);
  }
  // a wave without a place in the tile only fetches
  __device__ __forceinline__ void fetch_only() {
    for (int st = 0; st < nst; ++st) arrive(st);
  }
  // wm, wn: this wave's place
  __device__ __forceinline__ void run(const uint4* smem, int wm, int wn, f32x16 (&acc)[NB][1]) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][0][v] = 0.f;
    const uint4* mine = smem + (threadIdx.x & 63);
    int slot = 0;
    for (int st = 0; st < nst; ++st) {
      arrive(st);
      const uint4* buf = mine + (size_t)slot * (4 * F * 64);
      slot = slot + 1 == D ? 0 : slot + 1;
      Frag x[4], w[4][NB];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        x[h].u = buf[(h * F + wm) * 64];
#pragma unroll
        for (int b = 0; b < NB; ++b) w[h][b].u = buf[(h * F + FX + wn * NB + b) * 64];
      }
      __builtin_amdgcn_sched_barrier(0);   // all of a stage's reads are on their way before the first MFMA
#pragma unroll
      for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b][0] = mfma32(w[h][b], x[h], acc[b][0]);
    }
  }
};

// BIG_SWIGLU and BIG_ADD_F32 on tiles of 32 WM tokens x 64 WN features
template <int WM, int WN, int D, bool PK>
__global__ void __launch_bounds__(256, 2) k_gemm_mid(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, const int* rows, int M, int N,
                                                     int K, BigEpi ep) {
  extern __shared__ uint4 smem[];
  int bx, by;
  M = rows_there<PK>(rows, M);
  if (!big_raster(N / (64 * WN), (M + 32 * WM - 1) / (32 * WM), bx, by)) return;
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const bool live = wave < WM * WN;
  const int wm = live ? wave / WN : 0, wn = live ? wave % WN : 0;
  const int n0 = (bx * WN + wn) * 64;                    // the wave's first feature
  const int row0 = (by * WM + wm) * 32, tok = row0 + (lane & 31);
  f32x16 acc[2][1];
  float row_scale[1] = {1.f};
  {
    MidLoop<WM, WN, 2, D> loop;
    loop.begin(Xp, Wp, (M + 31) >> 5, K >> 4, by * WM, bx * WN * 2, smem);
    if (ep.ssq_in) row_scales<1>(ep.ssq_in, ep.ssq_parts, ep.ssq_halves, ep.norm_dim, ep.eps, tok, M, row_scale);
    if (live) loop.run(smem, wm, wn, acc);
    else loop.fetch_only();
  }
  if (!live) {
    if (ep.mode != BIG_SWIGLU) wg_barrier();
    return;
  }
  if (ep.ssq_in) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][0][v] *= row_scale[0];
  }
  if (ep.mode == BIG_SWIGLU) {
    if (tok >= M) return;
    const int F = N >> 1, f0 = (n0 >> 1) + (lane >> 5) * 4;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        f16x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = from_f32<f16>(silu_f(acc[b][0][4 * r + j]) * acc[b][0][4 * (r + 2) + j]);
        *(f16x4*)(ep.out_act + x32_chunk(tok, f0 + 16 * b + 8 * r, F >> 4) * 8 + ((lane >> 5) << 2)) = o;
      }
    return;
  }
  // BIG_ADD_F32: one pass of k_gemm_big's residual update (32 tokens x 64 features in row layout through LDS)
  wg_barrier();   // every wave has read its last stage: the ring is free
  if (row0 >= M) return;
  constexpr int RS = 68;
  float* R = (float*)smem + wave * (32 * RS);
  const int rt = lane >> 4, rc = (lane & 15) * 4;
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  float4 io[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)   // rows past the end: the last one again, not stored
    io[i] = *(const float4*)(ep.out_f32 + (size_t)min(row0 + 4 * i + rt, M - 1) * ep.ldc + n0 + rc);
  const bool prod = ep.gain_next != nullptr;
  float4 gn[2][4];
  if (prod) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) gn[b][r] = *(const float4*)(ep.gain_next + n0 + b * 32 + 8 * r + (lane >> 5) * 4);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) *(float4*)(R + (4 * i + rt) * RS + rc) = io[i];
  wave_sync();
  float ssq = 0.f;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float4* q = (float4*)(R + (lane & 31) * RS + b * 32 + 8 * r + (lane >> 5) * 4);
      const float4 w = *q;
      const float4 v = make_float4(acc[b][0][4 * r] + w.x, acc[b][0][4 * r + 1] + w.y, acc[b][0][4 * r + 2] + w.z,
                                   acc[b][0][4 * r + 3] + w.w);
      *q = v;
      if (prod && tok < M) {
        ssq += sum_squares4(v);
        f16x4 hv;
        hv[0] = from_f32<f16>(v.x * gn[b][r].x); hv[1] = from_f32<f16>(v.y * gn[b][r].y);
        hv[2] = from_f32<f16>(v.z * gn[b][r].z); hv[3] = from_f32<f16>(v.w * gn[b][r].w);
        *(f16x4*)(ep.xn_out + x32_chunk(tok, n0 + (lane >> 5) * 4 + b * 32 + 8 * r, N >> 4) * 8 + ((lane >> 5) << 2)) = hv;
      }
    }
  ssq += __shfl_xor(ssq, 32, 64);
  if (prod && lane < 32 && tok < M) ep.ssq_out[(size_t)tok * (((N >> 6) + 3) & ~3) + (n0 >> 6)] = ssq;
  wave_sync();
#pragma unroll
  for (int i = 0; i < 8; ++i) io[i] = *(const float4*)(R + (4 * i + rt) * RS + rc);
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (row0 + 4 * i + rt < M) *(float4*)(ep.out_f32 + (size_t)(row0 + 4 * i + rt) * ep.ldc + n0 + rc) = io[i];
}

// ---------------------------------------------------------------------------------------
// QKV projection with the rotary embedding and the KV append in its epilogue (token-parallel path): the
// fp32 q/k/v rows never exist in memory.  Same main loop as k_gemm_big.  A 128-feature tile is two heads of 64 (blocks
// 0, 1 and 2, 3) or one head of 128; the rotation partner (i + 32, resp. i + 64) sits in the same lane, one or two
// accumulator blocks on.  q goes out as half row-major [M, Hq hd] (flash attention's operand), rotated k and v go to the
// row's cache page.
// ---------------------------------------------------------------------------------------
// A wave's 64 tokens x 128 features of values, finished, into their V pages.  A lane's accumulators are features of one token,
// a page holds 8 tokens of a feature side by side: written from the registers that is two bytes per lane in runs of 16
// bytes, and the few workgroups with values end the launch.  They go through the wave's own LDS ([feature][token]) and leave
// as 16 bytes per lane wherever 8 slots are all here.  0.5B, 9 x 301 tokens: 21.1 us per launch; 31.4 with two bytes per lane
// (21.6 while a page held 16 tokens of a feature side by side, in runs of 32 bytes), 20.1 with the values' stores left
// out, 24.7 with 64 features at a time, twice the runs.
constexpr int kValueStride = 66;   // halves from a feature to the next: the lanes of a write and of a read are in different banks
constexpr int kQkvLds = 4 * 128 * kValueStride * (int)sizeof(f16);   // the ring is smaller; two workgroups fit a compute unit
static_assert(kQkvLds >= kBigLds && 2 * kQkvLds <= 160 * 1024, "ring, then the values of four waves");
template <int HD>
__device__ __forceinline__ void store_values(f32x16 (&acc)[4][2], const QkvEpi& ep, int head0, int row0, int M, const int (&pos_of)[2],
                                             const int (&page_of)[2], const bool (&keeps)[2], f16* area) {
  constexpr int RS = kValueStride;
  const int lane = threadIdx.x & 63, half_sel = lane >> 5, n_tok = min(64, M - row0);
  const int hkv = ep.kv.n_kv_heads;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        area[(b * 32 + 8 * (v >> 2) + (v & 3) + 4 * half_sel) * RS + tj * 32 + (lane & 31)] = from_f32<f16>(acc[b][tj][v]);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // features lane and lane + 64 of the tile: head f / HD, dim f % HD
  f16* vpool = (f16*)ep.kv.v + (size_t)(head0 - ep.n_q_heads - hkv) * HD * kPageTokens;
  const int at0 = (lane / HD) * HD * kPageTokens + v_page_at(0, lane % HD);
  const int at1 = ((lane + 64) / HD) * HD * kPageTokens + v_page_at(0, (lane + 64) % HD);
  const f16* src0 = area + lane * RS;
  const f16* src1 = src0 + 64 * RS;
  const unsigned long long kept[2] = {__builtin_amdgcn_ballot_w64(keeps[0]), __builtin_amdgcn_ballot_w64(keeps[1])};
  const unsigned long long kept64 = (kept[0] & 0xffffffffull) | (kept[1] << 32);   // bit t: token t stays in the cache
  const unsigned long long first64 = (__builtin_amdgcn_ballot_w64(pos_of[0] == 0) & 0xffffffffull) | (__builtin_amdgcn_ballot_w64(pos_of[1] == 0) << 32);
  // runs of tokens within 8 slots of a page; the lane that looked a token up knows its position and page
  for (int t = 0; t < n_tok;) {
    const int from = t & 31, pos = __builtin_amdgcn_readlane(t < 32 ? pos_of[0] : pos_of[1], from);
    const int page = __builtin_amdgcn_readlane(t < 32 ? page_of[0] : page_of[1], from);
    const unsigned long long next = t < 63 ? first64 >> (t + 1) : 0;   // bit i: token t + 1 + i is a sequence's first
    const int n = ep.rm.decode ? 1 : min(min(8 - (pos & 7), n_tok - t), next ? __builtin_ctzll(next) + 1 : 8);
    f16* dst = vpool + (size_t)page * hkv * HD * kPageTokens + v_page_at(pos % kPageTokens, 0);
    const unsigned stays = (unsigned)(kept64 >> t) & ((1u << n) - 1);
    if (stays == 0xff) {
      Frag o0, o1;
#pragma unroll
      for (int i = 0; i < 8; ++i) { o0.h[i] = src0[t + i]; o1.h[i] = src1[t + i]; }
      *(uint4*)(dst + at0) = o0.u;
      *(uint4*)(dst + at1) = o1.u;
    } else {
      for (int i = 0; i < n; ++i)
        if (stays >> i & 1) { dst[at0 + i] = src0[t + i]; dst[at1 + i] = src1[t + i]; }
    }
    t += n;
  }
}

// Of two groups of 4 values per lane, lanes l and l + 32 holding the first and the second half of 8: lane l's 8 of `a`, lane
// l + 32's 8 of `b`
__device__ __forceinline__ uint4 trade_halves(f16x4 a, f16x4 b) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 x = __builtin_bit_cast(u32x2, a), y = __builtin_bit_cast(u32x2, b);
  const u32x2 w0 = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false), w1 = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
  return make_uint4(w0[0], w1[0], w0[1], w1[1]);
}

// The epilogue of a wave's tile of NH heads, the first of them head0.  smem: the workgroup's ring (large tiles).  PK: packed rows (a
// kernel of its own: with both cases in one, the rotary pairs' loads waited for the page lookup, 1.2 us a layer).
template <int HD, int NH, int TJ, bool PK>
__device__ __forceinline__ void qkv_epilogue(f32x16 (&acc)[NH * (HD / 32)][TJ], const QkvEpi& ep, int head0, int tok0, int M,
                                             const float (&row_scale)[TJ], uint4* smem = nullptr) {
  constexpr int NB = HD / 32;   // accumulator blocks of a head
  const int lane = threadIdx.x & 63;
  const int hq = ep.n_q_heads, hkv = ep.kv.n_kv_heads;
  const int half_sel = lane >> 5;
  // row scale and bias first: what is rotated is the finished projection
#pragma unroll
  for (int fi = 0; fi < NH * NB; ++fi) {
    float4 bb[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      bb[r] = ep.bias ? *(const float4*)(ep.bias + head0 * HD + fi * 32 + half_sel * 4 + 8 * r) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[fi][tj][4 * r + 0] = acc[fi][tj][4 * r + 0] * row_scale[tj] + bb[r].x;
        acc[fi][tj][4 * r + 1] = acc[fi][tj][4 * r + 1] * row_scale[tj] + bb[r].y;
        acc[fi][tj][4 * r + 2] = acc[fi][tj][4 * r + 2] * row_scale[tj] + bb[r].z;
        acc[fi][tj][4 * r + 3] = acc[fi][tj][4 * r + 3] * row_scale[tj] + bb[r].w;
      }
  }
  f16* kpool = (f16*)ep.kv.k;
  f16* vpool = (f16*)ep.kv.v;
  // Where the token blocks of this lane go: position, cache page.  The page-table lookups are in flight together
  // (rows past the end look up row M - 1 and store nothing).
  int pos_of[TJ], page_of[TJ];
  bool keeps[TJ];
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) {
    const int tokc = min(tok0 + tj * 32, M - 1);
    keeps[tj] = ep.rm.keeps_kv(tokc);
    if constexpr (PK) {
      const int2 at = ep.rm.packed[tokc];
      page_of[tj] = at.x;
      pos_of[tj] = at.y;
    } else {
      int seq;
      ep.rm.get(tokc, seq, pos_of[tj]);
      page_of[tj] = ep.kv.page_table[(size_t)seq * ep.kv.pages_per_seq + pos_of[tj] / kPageTokens];
    }
  }
  const bool rotates = head0 < hq + hkv;   // else the tile is all V
  if constexpr (TJ == 2) {
    if (!rotates) {   // the same for the workgroup
      wg_barrier();   // nobody reads the ring any more
      store_values<HD>(acc, ep, head0, tok0 - (lane & 31), M, pos_of, page_of, keeps,
                       (f16*)smem + wave_index(threadIdx.x) * (kQkvLds / 4 / sizeof(f16)));
      return;
    }
  }
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) {
    const int tok = tok0 + tj * 32;
    // (cos, sin) of 32 of the block's pairs, the same for every head; the next ones (head dim 128) are requested before the
    // stores of what these gave: a load issued behind a store waits for the store's acknowledgement as well
    float4 cs[4][2];
    auto request = [&](int b) {
      const float2* cs_row = ep.rope + (size_t)pos_of[tj] * (HD / 2) + half_sel * 4;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        cs[r][0] = *(const float4*)(cs_row + b * 32 + 8 * r);
        cs[r][1] = *(const float4*)(cs_row + b * 32 + 8 * r + 2);
      }
    };
    if (rotates) request(0);
    if (tok >= M) continue;
#pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      const int head = head0 + hh;
      if (head >= hq && !keeps[tj]) continue;
      if (head >= hq + hkv) {
        const int vh = head - hq - hkv;
        // the lane's dims are 4 half_sel + a constant, which moves no carry in v_page_at: constant distances from its first one
        f16* vp = vpool + ((size_t)page_of[tj] * hkv + vh) * HD * kPageTokens + v_page_at(pos_of[tj] % kPageTokens, 4 * half_sel);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) vp[v_page_at(0, b * 32 + 8 * (v >> 2) + (v & 3))] = from_f32<f16>(acc[hh * NB + b][tj][v]);
        continue;
      }
      // the row's head, q row-major, k in its page (k_page_at), from the lane's 8 dims of each 16 on
      const bool is_q = head < hq;
      f16* dst = is_q ? ep.q_out + ((size_t)tok * hq + head) * HD + half_sel * 8
                      : kpool + ((size_t)page_of[tj] * hkv + (head - hq)) * kPageTokens * HD +
                            k_page_at(pos_of[tj] % kPageTokens, half_sel * 8);
#pragma unroll
      for (int b = 0; b < NB / 2; ++b) {
        f16x4 o1[4], o2[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float4 c01 = cs[r][0], c23 = cs[r][1];
          const float c[8] = {c01.x, c01.y, c01.z, c01.w, c23.x, c23.y, c23.z, c23.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float x1 = acc[hh * NB + b][tj][4 * r + j], x2 = acc[hh * NB + b + NB / 2][tj][4 * r + j];
            const float co = c[2 * j], sn = c[2 * j + 1];
            o1[r][j] = from_f32<f16>(rot_first(x1, x2, co, sn));
            o2[r][j] = from_f32<f16>(rot_second(x1, x2, co, sn));
          }
        }
        if (b + 1 < NB / 2) request(b + 1);
        // A lane holds dims 0 .. 3 or 4 .. 7 of every 8; two groups are traded with the lane that holds the others, so that each
        // stores 16 bytes (8 at a time the rows of q took twice the requests: 64 x 768 tokens at 0.5B 160 -> 149 us per launch).
        auto store = [&](auto at) {   // at(dim): where a dim lies behind the head's first one
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            *(uint4*)(dst + at(b * 32 + r * 8)) = trade_halves(o1[r], o1[r + 1]);
            *(uint4*)(dst + at((b + NB / 2) * 32 + r * 8)) = trade_halves(o2[r], o2[r + 1]);
          }
        };
        if (is_q) store([](int dim) { return dim; });
        else store([](int dim) { return k_page_at(0, dim); });
      }
    }
  }
}
template <int HD, int TJ, bool PK>
__global__ void __launch_bounds__(256, 2) k_gemm_qkv_rope(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, const int* rows, int M,
                                                          int N, int K, QkvEpi ep) {
  constexpr int H = 4, NH = 128 / HD, TM = 128 * TJ;   // heads and tokens of a tile
  extern __shared__ uint4 smem[];
  int bx, by;
  M = rows_there<PK>(rows, M);
  if (!big_raster(N >> 7, (M + TM - 1) / TM, bx, by)) return;
  f32x16 acc[4][TJ];
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const int tok0 = by * TM + wave * (32 * TJ) + (lane & 31);
  float row_scale[TJ];
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) row_scale[tj] = 1.f;
  {
    TileLoop<TJ, H> loop;
    loop.tokens(Xp, (M + 31) >> 5, K >> 4, by * (4 * TJ), 0);
    loop.features(Wp, K >> 4, bx * 4, 0, K / (16 * H), smem);
    loop.begin();
    if (ep.ssq_in) row_scales<TJ>(ep.ssq_in, ep.ssq_parts, ep.ssq_halves, ep.norm_dim, ep.eps, tok0, M, row_scale);
    loop.run(smem, acc);
  }
  qkv_epilogue<HD, NH, TJ, PK>(acc, ep, bx * NH, tok0, M, row_scale, smem);
}

// The same for few tokens: 32 WM tokens x one head per workgroup
template <int HD, int WM, int D, bool PK>
__global__ void __launch_bounds__(256, 2) k_gemm_qkv_mid(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, const int* rows, int M, int N,
                                                         int K, QkvEpi ep) {
  constexpr int NB = HD / 32;
  extern __shared__ uint4 smem[];
  int bx, by;
  M = rows_there<PK>(rows, M);
  if (!big_raster(N / HD, (M + 32 * WM - 1) / (32 * WM), bx, by)) return;
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const bool live = wave < WM;
  const int wm = live ? wave : 0, tok = (by * WM + wm) * 32 + (lane & 31);
  f32x16 acc[NB][1];
  float row_scale[1] = {1.f};
  MidLoop<WM, 1, NB, D> loop;
  loop.begin(Xp, Wp, (M + 31) >> 5, K >> 4, by * WM, bx * NB, smem);
  if (ep.ssq_in) row_scales<1>(ep.ssq_in, ep.ssq_parts, ep.ssq_halves, ep.norm_dim, ep.eps, tok, M, row_scale);
  if (!live) {
    loop.fetch_only();
    return;
  }
  loop.run(smem, wm, 0, acc);
  qkv_epilogue<HD, 1, 1, PK>(acc, ep, bx, tok, M, row_scale);
}

int n_compute_units() {
  static int n_cu = 0;
  if (n_cu == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      n = 256;
    n_cu = n;
  }
  return n_cu;
}
// SAPO_BIG_TILE=128 / 256 in the environment forces one of the large tiles (measurement, tests); read per call, so that a test
// can switch it
static int forced_tile() {
  const char* e = getenv("SAPO_BIG_TILE");
  const int t = e ? atoi(e) : 0;
  return t == 128 || t == 256 ? t : 0;
}
// Tiles for few tokens.  A workgroup's time is what it has to take in, so the tile is the one whose fullest compute unit
// takes in least: workgroups per unit x (tokens + features) of a tile; the large tiles' fetch (two stages ahead) counts
// half as much again, and a little more: two tiles of 64 x 128 on a unit are faster than one of 128 x 128 (scoring calls, us, 0.5B: 301
// tokens 1660 -> 1540, 2709 4024 -> 3767, 3600 4982 -> 4709; 1.5B: 128 tokens 2817 -> 2653, 1800 7570 -> 7156).  deep:
// one workgroup per unit, the whole LDS as its ring; otherwise two share it.
enum { MID_FFN, MID_QKV64, MID_QKV128 };
struct MidPick { int tile; bool deep; };   // tile: 0 = none of them, 1 = 32, 2 = 64 tokens x one wave's features, 3 = 64 x 128
static MidPick pick_mid(int M, int N, int what) {
  const int cu = n_compute_units(), nb = what == MID_QKV128 ? 128 : 64;
  auto groups = [&](int tm, int tn) { return (long)((M + tm - 1) / tm) * ((N + tn - 1) / tn); };
  auto load = [&](int tm, int tn, double weight) { return (double)((groups(tm, tn) + cu - 1) / cu) * (tm + tn) * weight; };
  MidPick best{0, true};
  if (forced_tile() != 0) return best;
  double least = std::min(load(256, 128, 1.55), what == MID_FFN ? load(128, 128, 1.55) : 1e30);
  const int tm[4] = {0, 32, 64, 64}, tn[4] = {0, nb, nb, 128};
  for (int t = 1; t <= (what == MID_FFN ? 3 : 2); ++t) {
    const long g = groups(tm[t], tn[t]);
    if (g > 2 * cu) continue;
    const double l = load(tm[t], tn[t], 1.0);
    if (l < least) { least = l; best.tile = t; best.deep = g <= cu; }
  }
  return best;
}
template <typename Kernel, typename Epi>
static hipError_t launch_mid(Kernel kernel, int lds, bool& attr_done, int grid, const uint4* X, const uint4* W, int M, int N, int K,
                             const Epi& epi, hipStream_t st) {
  if (!attr_done) {
    const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  return launch(KID_GEMM_BIG, kernel, dim3(grid), dim3(256), lds, st, X, W, epi.rows, M, N, K, epi);
}
template <int WM, int WN, int D>
static hipError_t launch_ffn_mid(const uint4* X, const uint4* W, int M, int N, int K, const BigEpi& epi, hipStream_t st) {
  static bool attr_done[2] = {false, false};
  static_assert(MidLoop<WM, WN, 2, D>::kBytes >= WM * WN * 32 * 68 * 4, "the residual update's row areas lie in the ring");
  const bool pk = epi.rows != nullptr;
  return launch_mid(pk ? k_gemm_mid<WM, WN, D, true> : k_gemm_mid<WM, WN, D, false>, MidLoop<WM, WN, 2, D>::kBytes, attr_done[pk], big_grid(N / (64 * WN), (M + 32 * WM - 1) / (32 * WM)),
                    X, W, M, N, K, epi, st);
}
template <int HD, int WM, int D>
static hipError_t launch_qkv_mid(const uint4* X, const uint4* W, int M, int N, int K, const QkvEpi& epi, hipStream_t st) {
  static bool attr_done[2] = {false, false};
  const bool pk = epi.rm.packed != nullptr;
  return launch_mid(pk ? k_gemm_qkv_mid<HD, WM, D, true> : k_gemm_qkv_mid<HD, WM, D, false>, MidLoop<WM, 1, HD / 32, D>::kBytes,
                    attr_done[pk], big_grid(N / HD, (M + 32 * WM - 1) / (32 * WM)), X, W, M, N, K, epi, st);
}
// 128-token instead of 256-token tiles by what the fullest compute unit multiplies, the smaller tile's operand traffic counted as
// 8 %.  Scoring calls, us with 256- and 128-token tiles of gate/up, 0.5B: 1600 tokens 2859, 2668; 1800 3060, 2983; 2250 3228, 3232 (6
// and 12 half tiles: equal); 3600 4992, 4924; 4800 5531, 5592; 6000 6599, 6500; 1.5B: 2709 10304, 10461; 4800 14370, 14729.  Of QKV,
// 0.5B: 1800 tokens 2950, 2792; 2250 3228, 3100; 2709 3738, 3628; 8100 7897, 7896; 1.5B, 4800 14566, 14389; where the rule keeps 256-token
// tiles, 0.5B: 12000 11060, 11123; 3600 4332, 4270; 6000 6379, 6334; 1.5B: 2709 9952, 9955; 3600 12117, 12021 (two half tiles on a unit
// take up to 1.4 % less of a call than one whole one here; the line is the one for both products).
static bool half_tiles_leave_less(int NX, int M) {
  const long cu = n_compute_units(), big = (long)NX * ((M + 255) / 256), small = (long)NX * ((M + 127) / 128);
  return (double)((small + cu - 1) / cu * 128) * 1.08 < (double)((big + cu - 1) / cu * 256);
}
bool m_gemm_writes_halves(int M, int N) { return pick_mid(M, N, MID_FFN).tile != 0; }
hipError_t m_gemm_qkv_rope(const void* Xp, const void* Wp, int M, int N, int K, const QkvEpi& epi, hipStream_t st) {
  if (M == 0) return hipSuccess;
  const int hd = epi.kv.head_dim;
  if (N % 128 != 0 || K % 64 != 0 || (hd != 64 && hd != 128) || N != (epi.n_q_heads + 2 * epi.kv.n_kv_heads) * hd)
    return hipErrorInvalidValue;
  {
    const MidPick m = pick_mid(M, N, hd == 64 ? MID_QKV64 : MID_QKV128);
    const uint4 *X = (const uint4*)Xp, *W = (const uint4*)Wp;
    if (hd == 64 && m.tile == 1) return m.deep ? launch_qkv_mid<64, 1, 10>(X, W, M, N, K, epi, st) : launch_qkv_mid<64, 1, 5>(X, W, M, N, K, epi, st);
    if (hd == 64 && m.tile == 2) return m.deep ? launch_qkv_mid<64, 2, 8>(X, W, M, N, K, epi, st) : launch_qkv_mid<64, 2, 4>(X, W, M, N, K, epi, st);
    if (hd == 128 && m.tile == 1) return m.deep ? launch_qkv_mid<128, 1, 7>(X, W, M, N, K, epi, st) : launch_qkv_mid<128, 1, 4>(X, W, M, N, K, epi, st);
    if (hd == 128 && m.tile == 2) return m.deep ? launch_qkv_mid<128, 2, 6>(X, W, M, N, K, epi, st) : launch_qkv_mid<128, 2, 3>(X, W, M, N, K, epi, st);
  }
  // With few workgroups the dispatcher may still put two on one compute unit, and the launch then takes their time one after the
  // other: 0.5B, 10 .. 16 token tiles, 20 us in some launches and 27 in most.  With more than half of a unit's LDS each has its
  // own: 39 x 64 tokens 26.6 -> 20.0, 64 x 64 28.5 -> 21.5 (at most 18 workgroups on the fullest XCD of 32 units).  At 27 on an XCD it
  // took 38.8 instead of 30.5, with a raster whose empty workgroups asked for the LDS too.
  constexpr int kAloneLds = 84 * 1024;
  static bool attr_done = false;
  if (!attr_done) {
    const auto with_lds = [](auto kernel, int lds) { return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds); };
    const auto both = [&](auto pk) {
      constexpr bool PK = decltype(pk)::value;
      hipError_t e = with_lds(k_gemm_qkv_rope<64, 2, PK>, kAloneLds);
      if (e == hipSuccess) e = with_lds(k_gemm_qkv_rope<128, 2, PK>, kAloneLds);
      if (e == hipSuccess) e = with_lds(k_gemm_qkv_rope<64, 1, PK>, kBigLds);
      return e == hipSuccess ? with_lds(k_gemm_qkv_rope<128, 1, PK>, kBigLds) : e;
    };
    hipError_t e = both(std::false_type());
    if (e == hipSuccess) e = both(std::true_type());
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int NX = N / 128, NY = (M + 255) / 256, per_xcd = (NX * NY + 7) / 8;
  auto go = [&](auto kernel, int ny, int lds) {
    return launch(KID_GEMM_BIG, kernel, dim3(big_grid(NX, ny)), dim3(256), lds, st, (const uint4*)Xp, (const uint4*)Wp, epi.rows, M, N, K, epi);
  };
  const auto pick = [&](auto pk) {
    constexpr bool PK = decltype(pk)::value;
    if (forced_tile() != 0 ? forced_tile() == 128 : half_tiles_leave_less(NX, M)) {
      const int ny = (M + 127) / 128;
      return hd == 64 ? go(k_gemm_qkv_rope<64, 1, PK>, ny, kBigLds) : go(k_gemm_qkv_rope<128, 1, PK>, ny, kBigLds);
    }
    const int lds = per_xcd <= 20 ? kAloneLds : kQkvLds;
    return hd == 64 ? go(k_gemm_qkv_rope<64, 2, PK>, NY, lds) : go(k_gemm_qkv_rope<128, 2, PK>, NY, lds);
  };
  return epi.rm.packed ? pick(std::true_type()) : pick(std::false_type());
}

// 128-token tiles (three workgroups per compute unit) instead of 256-token tiles (two): for narrow outputs whose
// 256-token tiles fill their last round of resident workgroups badly, when the half-size tiles need no more rounds
// (64 x 384 tokens x 896 features: 672 tiles in 2 rounds of 512 become 1344 in 2 rounds of 768; O projection 86 ->
// 70 us, the prompt's small launches 70 -> 58 us.  With one round more - 64 x 768: 4 against 3 - the down projection
// lost 14 %, so that case keeps the large tile).
static bool big_prefers_small_tiles(int NX, int M) {
  const int n_cu = n_compute_units();
  if (forced_tile() != 0) return forced_tile() == 128;
  if (NX > 16) return half_tiles_leave_less(NX, M);
  const long big = (long)NX * ((M + 255) / 256), small = (long)NX * ((M + 127) / 128);
  const long rounds_big = (big + 2 * n_cu - 1) / (2 * n_cu), rounds_small = (small + 3 * n_cu - 1) / (3 * n_cu);
  return rounds_small <= rounds_big;
}

template <int TJ, int H, int MODE>
static hipError_t launch_big(const void* Xp, const void* Wp, int M, int N, int K, const BigEpi& epi, hipStream_t st) {
  static bool attr_done[2] = {false, false};
  const bool pk = epi.rows != nullptr;
  const auto kernel = pk ? k_gemm_big<TJ, H, MODE, true> : k_gemm_big<TJ, H, MODE, false>;
  // the residual update's four row areas and gains lie in the ring's memory
  constexpr int lds = ring_bytes(H) > 4 * (32 * 68 + 128) * 4 ? ring_bytes(H) : 4 * (32 * 68 + 128) * 4;
  if (!attr_done[pk]) {
    const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_done[pk] = true;
  }
  return launch(KID_GEMM_BIG, kernel, dim3(big_grid(N / 128, (M + 128 * TJ - 1) / (128 * TJ))), dim3(256), lds, st,
                (const uint4*)Xp, (const uint4*)Wp, epi.rows, M, N, K, epi);
}
template <int TJ, int H>
static hipError_t launch_big(const void* Xp, const void* Wp, int M, int N, int K, const BigEpi& epi, hipStream_t st) {
  if (epi.mode == BIG_SWIGLU) return launch_big<TJ, H, BIG_SWIGLU>(Xp, Wp, M, N, K, epi, st);
  if (epi.mode == BIG_ADD_F32) return launch_big<TJ, H, BIG_ADD_F32>(Xp, Wp, M, N, K, epi, st);
  return launch_big<TJ, H, BIG_STORE_F32>(Xp, Wp, M, N, K, epi, st);
}
hipError_t m_gemm_big(const void* Xp, const void* Wp, int M, int N, int K, BigEpi epi, hipStream_t st) {
  if (M == 0) return hipSuccess;
  if (N % 128 != 0 || K % 64 != 0) return hipErrorInvalidValue;
  if ((epi.gain_next && epi.mode != BIG_ADD_F32) || (epi.ssq_in && epi.mode == BIG_ADD_F32)) return hipErrorInvalidValue;
  if (epi.mode != BIG_STORE_F32) {
    const MidPick m = pick_mid(M, N, MID_FFN);
    const uint4 *X = (const uint4*)Xp, *W = (const uint4*)Wp;
    if (m.tile == 1) return m.deep ? launch_ffn_mid<1, 1, 10>(X, W, M, N, K, epi, st) : launch_ffn_mid<1, 1, 5>(X, W, M, N, K, epi, st);
    if (m.tile == 2) return m.deep ? launch_ffn_mid<2, 1, 8>(X, W, M, N, K, epi, st) : launch_ffn_mid<2, 1, 4>(X, W, M, N, K, epi, st);
    if (m.tile == 3) return m.deep ? launch_ffn_mid<2, 2, 6>(X, W, M, N, K, epi, st) : launch_ffn_mid<2, 2, 3>(X, W, M, N, K, epi, st);
  }
  if (big_prefers_small_tiles(N / 128, M)) return launch_big<1, 4>(Xp, Wp, M, N, K, epi, st);
  return launch_big<2, 4>(Xp, Wp, M, N, K, epi, st);
}

// ---------------------------------------------------------------------------------------
// RMSNorm of residual rows into X32 order: out[i] = half( h[r] * rsqrt(mean(h[r]^2) + eps) * gain ),
// r = row_index ? row_index[i] : i; negative r (padding) gives zeros.  One workgroup per row.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(128) k_rmsnorm_x32(const float* __restrict__ h, const float* __restrict__ gain, float eps,
                                                     uint4* __restrict__ out, int d, const int* __restrict__ row_index,
                                                     const int* rows) {
  __shared__ float red[2];
  const int i = blockIdx.x;
  if (rows && i >= rows_there<true>(rows, gridDim.x)) return;
  const int r = row_index ? row_index[i] : i;
  const int KS = d >> 4;
  if (r < 0) {
    for (int k = threadIdx.x * 8; k < d; k += 1024) out[x32_chunk(i, k, KS)] = make_uint4(0, 0, 0, 0);
    return;
  }
  const float* x = h + (size_t)r * d;
  float ss = 0.f;
  for (int k = threadIdx.x * 4; k < d; k += 512) {
    const float4 v = *(const float4*)(x + k);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  ss = wave_reduce_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float scale = 1.0f / sqrtf((red[0] + red[1]) / (float)d + eps);
  for (int k = threadIdx.x * 8; k < d; k += 1024) {
    const float4 a = *(const float4*)(x + k), b = *(const float4*)(x + k + 4);
    const float4 ga = *(const float4*)(gain + k), gb = *(const float4*)(gain + k + 4);
    Frag o;
    o.h[0] = from_f32<f16>(a.x * scale * ga.x); o.h[1] = from_f32<f16>(a.y * scale * ga.y);
    o.h[2] = from_f32<f16>(a.z * scale * ga.z); o.h[3] = from_f32<f16>(a.w * scale * ga.w);
    o.h[4] = from_f32<f16>(b.x * scale * gb.x); o.h[5] = from_f32<f16>(b.y * scale * gb.y);
    o.h[6] = from_f32<f16>(b.z * scale * gb.z); o.h[7] = from_f32<f16>(b.w * scale * gb.w);
    out[x32_chunk(i, k, KS)] = o.u;
  }
}
hipError_t m_rmsnorm_x32(const float* h, const float* gain, float eps, void* out, int M, int d, const int* row_index,
                         hipStream_t st, const int* rows) {
  if (M == 0) return hipSuccess;
  return launch(KID_RMSNORM, k_rmsnorm_x32, dim3(M), dim3(128), 0, st, h, gain, eps, (uint4*)out, d, row_index, rows);
}

__global__ void __launch_bounds__(256) k_gather_rows_x32(const int* __restrict__ src_rows, const int* __restrict__ n_rows,
                                                         const float* __restrict__ h, int d, const uint4* __restrict__ x, int q,
                                                         float* __restrict__ h_out, uint4* __restrict__ x_out) {
  const int i = blockIdx.x;
  if (n_rows && i >= rows_there<true>(n_rows, gridDim.x)) return;
  const int r = src_rows[i];
  for (int k = threadIdx.x * 4; k < d; k += 1024) *(float4*)(h_out + (size_t)i * d + k) = *(const float4*)(h + (size_t)r * d + k);
  for (int k = threadIdx.x * 8; k < q; k += 2048) x_out[x32_chunk(i, k, q >> 4)] = x[x32_chunk(r, k, q >> 4)];
}
hipError_t m_gather_rows_x32(const int* src_rows, const int* n_rows, int M, const float* h, int d, const void* x, int q, float* h_out,
                             void* x_out, hipStream_t st) {
  if (M == 0) return hipSuccess;
  return launch(KID_MISC, k_gather_rows_x32, dim3(M), dim3(256), 0, st, src_rows, n_rows, h, d, (const uint4*)x, q, h_out, (uint4*)x_out);
}

// ---------------------------------------------------------------------------------------
// LM head for scoring: log-softmax + target gather without materialising logits.
// Rastered like the GEMM over (256-row tiles) x (groups of 128-feature tiles): a workgroup
// walks the tiles of its group for its 256 rows, leaves every tile's (max, sum exp) of every row, and the
// one lane that sees a row's target id writes the target logit.  A second kernel merges a row's tiles
// in one order, so that a log-prob has the same bits whatever else is scored: groups follow the number of scored rows, and with a
// (max, sum exp) per group a sequence's last bits changed with other sequences' masks.  32768 rows, vocabulary of 151936: 7.74 ms
// and 62 us for the merge; with groups as the unit, whose running maxima cost 4 more exponentials per lane and tile, 7.71 and 14.  2678
// rows: 507 and 8 us; 506 and 4.  (Blocks of two or three tiles as the unit: 3 .. 5 % longer, groups of whole blocks fill rounds worse.)
// partials: ztarget [max_rows], from the next even number on [tiles][n_rows][2].
// ---------------------------------------------------------------------------------------
static int score_slots() { return 2 * n_compute_units(); }   // workgroups in flight
__host__ __device__ constexpr size_t score_pairs_at(int max_rows) { return ((size_t)max_rows + 1) & ~(size_t)1; }
size_t m_lmhead_score_partial_floats(int max_rows, int V) { return score_pairs_at(max_rows) + 2 * (size_t)(V >> 7) * max_rows; }

__global__ void __launch_bounds__(256, 2) k_lmhead_score(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp,
                                                         int max_rows, const int* __restrict__ n_rows_dev, int V, int K,
                                                         const int* __restrict__ row_seq_pos,
                                                         const int32_t* __restrict__ tokens, int T, int slots,
                                                         float* __restrict__ partials) {
  constexpr int TJ = 2, H = 4;
  extern __shared__ uint4 smem[];
  const int n_rows = *n_rows_dev;
  const int n_ft = V >> 7;
  const int row_tiles = (n_rows + 255) >> 8;
  const ScoreGroups g(n_ft, row_tiles, slots);
  int bx, by;
  if (!big_raster(g.groups, row_tiles, bx, by)) return;
  const int ft_begin = bx * g.tiles, ft_end = min(n_ft, ft_begin + g.tiles);
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const int row0 = by * 256 + wave * 64 + (lane & 31);
  int target[TJ];
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) {
    const int row = row0 + tj * 32;
    target[tj] = -1;
    if (row < n_rows) target[tj] = tokens[(size_t)row_seq_pos[2 * row] * T + row_seq_pos[2 * row + 1]];
  }
  float2* const pairs = (float2*)(partials + score_pairs_at(max_rows));
  const int own_row = by * 256 + wave * 64 + lane;   // lane 32 and up: the row of tj 1
  float* ztarget = partials;
  TileLoop<TJ, H> loop;
  loop.tokens(Xp, (n_rows + 31) >> 5, K >> 4, by * 8, 0);
  loop.features(Wp, K >> 4, ft_begin * 4, 0, K / (16 * H), smem);
  loop.begin();
  for (int ft = ft_begin; ft < ft_end; ++ft) {
    f32x16 acc[4][TJ];
    loop.run(smem, acc);
    if (ft + 1 < ft_end) {   // the next tile's first stages are on their way during this tile's exponentials
      wg_barrier();          // every wave has read its last stage
      loop.features(Wp, K >> 4, (ft + 1) * 4, 0, K / (16 * H), smem);
      loop.begin();
    }
    float m[TJ], l[TJ];
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj) {
      float mt = acc[0][tj][0];
#pragma unroll
      for (int fi = 0; fi < 4; ++fi)
#pragma unroll
        for (int v = 0; v < 16; ++v) mt = fmaxf(mt, acc[fi][tj][v]);
      mt = max_xor32(mt);
      float su[4];
#pragma unroll
      for (int fi = 0; fi < 4; ++fi) {
        const int f0 = ft * 128 + fi * 32 + (lane >> 5) * 4;
        su[fi] = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) su[fi] += __expf(acc[fi][tj][v] - mt);
        const int dt = target[tj] - f0;   // target among this lane's 4 x 4 features?
        if (dt >= 0 && dt < 32 && (dt & 4) == 0) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (dt == 8 * (v >> 2) + (v & 3)) ztarget[row0 + tj * 32] = acc[fi][tj][v];
        }
      }
      m[tj] = mt;
      l[tj] = sum_xor32((su[0] + su[1]) + (su[2] + su[3]));   // in both halves of the wave
    }
    if (own_row < n_rows) pairs[(size_t)ft * n_rows + own_row] = make_float2(lane < 32 ? m[0] : m[1], lane < 32 ? l[0] : l[1]);
  }
}

// 16 rows per workgroup: thread (row, part) merges the tiles part, part + 64, ... in order, then the parts pairwise (16 parts: 10 us
// instead of 5 with few rows).
constexpr int kMergeThreads = 1024;
__global__ void __launch_bounds__(kMergeThreads) k_lmhead_score_merge(const float* __restrict__ partials, int max_rows, int V,
                                                                      const int* __restrict__ n_rows_dev, const int* __restrict__ row_seq_pos,
                                                                      int T, float* __restrict__ out_logprobs) {
  constexpr int kParts = kMergeThreads / 16;
  __shared__ float2 s_ml[kMergeThreads / 64][16];
  const int n_rows = *n_rows_dev, wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  if ((int)blockIdx.x * 16 >= n_rows) return;
  const int row = min((int)blockIdx.x * 16 + (lane & 15), n_rows - 1), n_tiles = V >> 7;
  const float2* p = (const float2*)(partials + score_pairs_at(max_rows)) + row;
  LseAcc a; a.init();
  auto over_parts = [&] {   // of the wave's four
#pragma unroll
    for (int o = 32; o >= 16; o >>= 1) a.merge(__shfl_xor(a.m, o, 64), __shfl_xor(a.l, o, 64));
  };
#pragma unroll 4
  for (int s = threadIdx.x >> 4; s < n_tiles; s += kParts) {
    const float2 ml = p[(size_t)s * n_rows];
    a.merge(ml.x, ml.y);
  }
  over_parts();
  if (lane < 16) s_ml[wave][lane] = make_float2(a.m, a.l);
  __syncthreads();
  if (wave != 0) return;
  a.init();
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float2 ml = s_ml[(lane >> 4) * 4 + w][lane & 15];
    a.merge(ml.x, ml.y);
  }
  over_parts();
  if (lane >= 16 || (int)blockIdx.x * 16 + lane >= n_rows) return;
  const float zt = partials[row];
  out_logprobs[(size_t)row_seq_pos[2 * row] * T + row_seq_pos[2 * row + 1]] = zt - (a.m + logf(a.l));
}

hipError_t m_lmhead_score(const void* Xp, const void* Wp, int max_rows, const int* n_rows_dev, int V, int K,
                          const int* row_seq_pos, const int32_t* tokens, int T, float* partials, float* out_logprobs,
                          hipStream_t st) {
  if (max_rows == 0) return hipSuccess;
  if (V % 128 != 0 || K % 64 != 0) return hipErrorInvalidValue;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)k_lmhead_score, hipFuncAttributeMaxDynamicSharedMemorySize, kBigLds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int slots = score_slots();
  const unsigned blocks = (unsigned)((score_most_workgroups(V >> 7, max_rows, slots) + 7) / 8 * 8);
  const hipError_t e = launch(KID_LMHEAD_SCORE, k_lmhead_score, dim3(blocks), dim3(256), kBigLds, st, (const uint4*)Xp,
                              (const uint4*)Wp, max_rows, n_rows_dev, V, K, row_seq_pos, tokens, T, slots, partials);
  if (e != hipSuccess) return e;
  return launch(KID_LMHEAD_SCORE_MERGE, k_lmhead_score_merge, dim3((max_rows + 15) / 16), dim3(kMergeThreads), 0, st, partials,
                max_rows, V, n_rows_dev, row_seq_pos, T, out_logprobs);
}

// ---------------------------------------------------------------------------------------
// LM head for decode with many sequences (or a K too large for the 64-token kernel): the scoring
// GEMM's main loop with the sampler's epilogue, one (256 or 128 sequences x 128 vocabulary ids) tile per
// workgroup.  A lane turns its quads of consecutive vocabulary ids into perturbed scores (one Philox
// block per quad) and reduces, for each of its sequences, (max, sum exp) and the best perturbed
// score.  partials: [V / 128][n_rows][5].
// ---------------------------------------------------------------------------------------
int m_lmhead_sample_big_groups(int V) { return V >> 7; }

template <int TJ>
__global__ void __launch_bounds__(256, TJ == 2 ? 2 : 3) k_lmhead_sample_big(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp,
                                                                            int n_rows, int V, int K, SampleParams sp,
                                                                            float* __restrict__ partials) {
  constexpr int H = 4, TM = 128 * TJ, RW = 32 * TJ;   // rows of a tile and of a wave
  extern __shared__ uint4 smem[];
  int ft, by;
  if (!big_raster(V >> 7, (n_rows + TM - 1) / TM, ft, by)) return;
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  f32x16 acc[4][TJ];
  {
    TileLoop<TJ, H> loop;
    loop.tokens(Xp, (n_rows + 31) >> 5, K >> 4, by * (TM / 32), 0);
    loop.features(Wp, K >> 4, ft * 4, 0, K / (16 * H), smem);
    if (by * TM + wave * RW >= n_rows) {   // no row of this wave exists
      loop.template begin<false>();
      loop.template run<false>(smem, acc);
      return;
    }
    loop.begin();
    loop.run(smem, acc);
  }
  resolve_sample_params(sp);
  const int step = *sp.step;
  const bool noisy = sp.temperature != 0.f;
  const float inv_t = noisy ? 1.0f / sp.temperature : 1.0f;
#pragma unroll
  for (int tj = 0; tj < TJ; ++tj) {
    const int row = by * TM + wave * RW + tj * 32 + (lane & 31);
    if (by * TM + wave * RW + tj * 32 >= n_rows) break;   // a whole block past the end
    const int seq = (sp.slot_seq && row < n_rows) ? sp.slot_seq[row] : row;   // the noise is keyed on the sequence
    LseAcc lse;
    BestAcc best;
    lse.init();
    best.init();
#pragma unroll
    for (int fi = 0; fi < 4; ++fi) {
      float mt = acc[fi][tj][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) mt = fmaxf(mt, acc[fi][tj][v]);
      const float mn = fmaxf(lse.m, mt);
      float su = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) su += __expf(acc[fi][tj][v] - mn);
      lse.l = lse.l * __expf(lse.m - mn) + su;
      lse.m = mn;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int v0 = ft * 128 + fi * 32 + 8 * r + (lane >> 5) * 4;
        float gn[4] = {0.f, 0.f, 0.f, 0.f};
        if (noisy) gumbel4(sp.seed_lo, sp.seed_hi, (uint32_t)seq, (uint32_t)step, (uint32_t)(v0 >> 2), gn);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float z = acc[fi][tj][4 * r + j];
          const float y = noisy ? z * inv_t + gn[j] : z;
          if (y > best.y) { best.y = y; best.z = z; best.id = v0 + j; }   // ids ascend within a lane
        }
      }
    }
    // the two lane halves (fixed order)
    lse.merge(__shfl_xor(lse.m, 32, 64), __shfl_xor(lse.l, 32, 64));
    best.add(__shfl_xor(best.y, 32, 64), __shfl_xor(best.z, 32, 64), __shfl_xor(best.id, 32, 64));
    if (lane < 32 && row < n_rows) {
      float* p = partials + ((size_t)ft * n_rows + row) * 5;
      p[0] = lse.m; p[1] = lse.l; p[2] = best.y; p[3] = best.z; ((int*)p)[4] = best.id;
    }
  }
}

hipError_t m_lmhead_sample_big(const void* Xp, const void* Wp, int n_rows, int V, int K, SampleParams sp, float* partials,
                               hipStream_t st) {
  if (n_rows <= 0 || V % 128 != 0 || K % 64 != 0) return hipErrorInvalidValue;
  auto go = [&](auto kernel, int rows, bool& attr_done) {
    if (!attr_done) {
      const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kBigLds);
      if (e != hipSuccess) return e;
      attr_done = true;
    }
    return launch(KID_LMHEAD_SAMPLE, kernel, dim3(big_grid(V >> 7, (n_rows + rows - 1) / rows)), dim3(256), kBigLds, st, (const uint4*)Xp,
                  (const uint4*)Wp, n_rows, V, K, sp, partials);
  };
  static bool done_128 = false, done_256 = false;
  // Up to 128 rows as 32 per wave: in the tile of 256 half the waves, always the same SIMDs', would have no row.
  // us per step, 0.5B: 72 rows 909 -> 898, 128 957 -> 938; 1.5B: 16 rows 1196 -> 1193,
  // 64 1624 -> 1609, 128 1699 -> 1683; the same bits.
  if (n_rows <= 128) return go(k_lmhead_sample_big<1>, 128, done_128);
  return go(k_lmhead_sample_big<2>, 256, done_256);
}

// =======================================================================================
// Causal GQA attention for prefill and scoring (many positions per sequence), MFMA 16x16x32.
// grid (sequences x KV heads; groups of HPW query heads; 64-position blocks), the longest walks of all sequences first: with
// the blocks fastest the compute units had waves 71 % of the time.
// A wave owns 16 query positions and up to HPW query heads that share the KV head, and walks the
// keys 0 .. last query position in 32-key page pairs read straight from the paged cache into
// fragment registers: S^T = K Q^T puts one query column in each lane, so the running max / sum are
// per-lane scalars (plus two shuffles) and the probabilities a lane produces are its operand of
// O^T = V^T P^T; key rows are permuted inside a pair so that a lane's 8 probabilities are 8
// consecutive tokens, what a lane gets from a V page in one 16-byte load (v_page_at).  No LDS, no
// block-level synchronisation; waves never exchange data.  q (row-major [rows, Hq hd]), K, V and the
// probabilities are IEEE half; the output goes out as half in X32 order (the O projection's operand).
// What bounds it: a SIMD issues MFMAs, vector instructions and (quarter rate) exponentials one after the other, 8 + ~35 + 8 per
// head and page pair, and their serial sum is the time.  So what could go went: the cross-lane maximum and the rescaling
// where no lane has a score above its query's maximum, register copies between the two page pairs in flight, page numbers
// as vector loads, operand quieting; the arithmetic is the same to the bit.  us per launch before and now: 64 x 768
// tokens, 14 heads of 64 198 -> 129, 12 heads of 128 322 -> 227; 9 x 301 tokens 15.0 -> 9.4.  (A reference that follows the
// maximum only in steps of more than 2^8 gives 115, 206 and 8.9, and other last bits.)
// ---------------------------------------------------------------------------------------
// The largest of a lane's 8 scores, two accumulators of 4, in 4 instructions (fmaxf() quiets the results of MFMAs first, which
// are not known to be free of signalling NaNs: 11).  The first one is the compiler's and reads both accumulators, so that
// the wait states behind the MFMAs have passed before the asm, which it knows nothing about; inf: +infinity in a register
// that it cannot see through.  A NaN score reaches the result through its own exponential whatever is found here.
__device__ __forceinline__ float max8(const float (&p)[8], float inf) {
  float m = __builtin_amdgcn_fmed3f(p[3], p[7], inf);
  asm("v_max3_f32 %0, %0, %1, %2\n\tv_max3_f32 %0, %0, %3, %4\n\tv_max3_f32 %0, %0, %5, %6"
      : "+v"(m) : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[4]), "v"(p[5]), "v"(p[6]));
  return m;
}
// the largest of lanes l, l ^ 16, l ^ 32 and l ^ 48, without quieting either
__device__ __forceinline__ float max_lanes(float x, float inf) {
  lane_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __builtin_amdgcn_fmed3f(__uint_as_float(r[0]), __uint_as_float(r[1]), inf);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __builtin_amdgcn_fmed3f(__uint_as_float(r[0]), __uint_as_float(r[1]), inf);
}

template <int HD, int HPW, bool PK>   // PK: packed rows
__global__ void __launch_bounds__(256, 2) k_flash_attention(const f16* __restrict__ q, RowMap rm, KVCache kv,
                                                         f16* __restrict__ out, int n_q_heads) {
  constexpr int KK = HD / 32, DT = HD / 16;
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const int qcol = lane & 15, grp = lane >> 4;
  const int qb = gridDim.z - 1 - blockIdx.z;   // the longest walks first, over all sequences
  const int hkv = kv.n_kv_heads, rep = n_q_heads / hkv;
  const int sblk = blockIdx.x / hkv, kvh = blockIdx.x % hkv;
  // read through the constant address space: scalar loads, which do not queue behind the K / V fragments
  typedef const __attribute__((address_space(4))) int* ConstInts;
  const ConstInts first = (ConstInts)rm.first;
  const size_t row0 = PK ? (size_t)first[sblk] : (size_t)sblk * rm.T;
  const int T = PK ? first[sblk + 1] - (int)row0 : rm.T;   // rows of the sequence
  const int h0 = blockIdx.y * HPW;
  const int nh = min(HPW, rep - h0);
  const int q0 = qb * 64 + wave * 16;
  if (q0 >= T) return;
  const ConstInts pt = (ConstInts)(kv.page_table + (size_t)(sblk * rm.seq_stride) * kv.pages_per_seq);
  const int qpos = min(q0 + qcol, T - 1);   // columns past T repeat the last position and are not stored
  const size_t qstride = (size_t)n_q_heads * HD;
  Frag qf[HPW][KK];
#pragma unroll
  for (int h = 0; h < HPW; ++h)
    if (h < nh) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        qf[h][kk].u = *(const uint4*)(q + (row0 + qpos) * qstride + (size_t)(kvh * rep + h0 + h) * HD + kk * 32 + grp * 8);
    }
  const float scale2 = 1.4426950408889634f / sqrtf((float)HD);   // scores in units of log2
  float inf = INFINITY;
  asm("" : "+s"(inf));
  float m_run[HPW], l_run[HPW];
  f32x4 o[HPW][DT];
#pragma unroll
  for (int h = 0; h < HPW; ++h) {
    m_run[h] = -INFINITY; l_run[h] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[h][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int q_hi = min(q0 + 15, T - 1);
  const int npairs = q_hi / 32 + 1;
  const int last_page = q_hi / kPageTokens;
  const size_t page_bytes = (size_t)hkv * kPageTokens * HD * sizeof(f16);
  const char* kpool = (const char*)kv.k + (size_t)kvh * kPageTokens * HD * sizeof(f16);
  const char* vpool = (const char*)kv.v + (size_t)kvh * kPageTokens * HD * sizeof(f16);
  const unsigned k_off = k_frag_at(0, 0, lane) * sizeof(f16), v_off = v_frag_at(0, lane) * sizeof(f16);
  const bool k_first = (lane & 15) < 8, v_first = grp < 2;
  // K / V fragments of a page pair; the next pair's are requested before the current one is multiplied (a third
  // register set, two pairs ahead, was measured at head dim 64: 238 against 223 us per launch at 64 x 768)
  Frag kf[2][2][KK], vf[2][DT];
  auto fetch = [&](int pp, auto buf) {
    constexpr int b = decltype(buf)::value;
    const size_t pa = (size_t)pt[2 * pp] * page_bytes, pb = (size_t)pt[min(2 * pp + 1, last_page)] * page_bytes;
    const char* kp = kpool + (k_first ? pa : pb) + k_off;
    const char* vp = vpool + (v_first ? pa : pb) + v_off;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        kf[b][t][kk].u = *(const uint4*)(kp + (k_frag_at(t, kk, 0) - k_frag_at(0, 0, 0)) * sizeof(f16));
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[b][dt].u = *(const uint4*)(vp + (v_frag_at(dt, 0) - v_frag_at(0, 0)) * sizeof(f16));
  };
  // DIAG: the walk's last pair, the only one with masked (query, key)s
  auto multiply = [&](int pp, auto buf, auto diag) {
    constexpr int b = decltype(buf)::value;
    constexpr bool DIAG = decltype(diag)::value;
#pragma unroll
    for (int h = 0; h < HPW; ++h) {
      if (h >= nh) break;
      f32x4 sc[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) sc[t] = mfma16h(kf[b][t][kk], qf[h][kk], sc[t]);
      }
      // lane (query qcol, group grp) holds keys pp*32 + 8 grp + e, e = 4 t + j
      float p[8];   // raw scores; the softmax scale enters through the exponent's fma
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = sc[e >> 2][e & 3];
      if constexpr (DIAG) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (pp * 32 + 8 * grp + e > qpos) p[e] = -INFINITY;
      }
      float m_loc = max8(p, inf) * scale2, alpha = 1.f;
      if (__builtin_amdgcn_ballot_w64(m_loc > m_run[h]) != 0) {   // the running maximum moves for some query
        asm volatile("");   // a branch: as selects, its 28 instructions would run for every pair
        m_loc = max_lanes(m_loc, inf);
        const float m_new = __builtin_amdgcn_fmed3f(m_run[h], m_loc, inf);   // finite: key 0 is visible to every query
        alpha = __builtin_amdgcn_exp2f(m_run[h] - m_new);   // exp2(-inf) = 0 on the first pair
        m_run[h] = m_new;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int j = 0; j < 4; ++j) o[h][dt][j] *= alpha;
      }
      float psum = 0.f;
      Frag pf;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pe = __builtin_amdgcn_exp2f(fmaf(p[e], scale2, -m_run[h]));
        psum += pe;
        pf.h[e] = (f16)pe;
      }
      l_run[h] = fmaf(l_run[h], alpha, psum);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[h][dt] = mfma16h(vf[b][dt], pf, o[h][dt]);
    }
  };
  const std::integral_constant<int, 0> even;
  const std::integral_constant<int, 1> odd;
  const std::true_type last;
  const std::false_type inner;
  // the requests of the loop sit under no branch: behind one, the compiler would wait for everything in flight
  fetch(0, even);
  int pp = 0;
  for (; pp + 2 < npairs; pp += 2) {
    fetch(pp + 1, odd);
    multiply(pp, even, inner);
    fetch(pp + 2, even);
    multiply(pp + 1, odd, inner);
  }
  if (pp + 1 < npairs) {
    fetch(pp + 1, odd);
    multiply(pp, even, inner);
    // copied, once per walk: a second copy of the masked code spilled registers (head dim 128, two heads)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[0][t][kk] = kf[1][t][kk];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[0][dt] = vf[1][dt];
    ++pp;
  }
  multiply(pp, even, last);
  if (q0 + qcol >= T) return;
#pragma unroll
  for (int h = 0; h < HPW; ++h) {
    if (h >= nh) continue;
    float l = l_run[h];
    l = sum_xor16(l);
    l = sum_xor32(l);
    const float inv = 1.0f / l;
    const int col0 = (kvh * rep + h0 + h) * HD + grp * 4;   // lane's 4 consecutive head dims, per 16-row tile
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      f16x4 ov;
#pragma unroll
      for (int j = 0; j < 4; ++j) ov[j] = from_f32<f16>(o[h][dt][j] * inv);
      const int col = col0 + dt * 16;
      *(f16x4*)(out + x32_chunk((int)row0 + qpos, col, (int)(qstride >> 4)) * 8 + (col & 4)) = ov;
    }
  }
}

hipError_t m_flash_attention(const void* q, RowMap rm, KVCache kv, void* out, int n_seq, int n_q_heads, hipStream_t st) {
  if (n_seq == 0) return hipSuccess;
  const int rep = n_q_heads / kv.n_kv_heads;
  const int nqb = (rm.T + 63) / 64;
  // Query heads per wave.  4 at head dim 64 (2 at 128): a 7-head group goes to two workgroups (4 + 3 heads): two waves per
  // SIMD, which hide the softmax arithmetic, pay for the second read of K / V.  With few sequences a wave's walk over the
  // keys is what the launch takes, and fewer heads shorten it: the most that still leave a workgroup for every compute unit.
  auto go = [&](auto kernel, int hpw) {
    return launch(KID_FLASH_ATTN, kernel, dim3(n_seq * kv.n_kv_heads, (rep + hpw - 1) / hpw, nqb), dim3(256), 0, st, (const f16*)q, rm,
                  kv, (f16*)out, n_q_heads);
  };
  auto groups = [&](int hpw) { return (long)nqb * n_seq * kv.n_kv_heads * ((rep + hpw - 1) / hpw); };
  const long cu = n_compute_units();
  const auto pick = [&](auto pk) {
    constexpr bool PK = decltype(pk)::value;
    if (kv.head_dim == 64) {
      if (groups(4) >= cu) return go(k_flash_attention<64, 4, PK>, 4);
      if (groups(2) >= cu) return go(k_flash_attention<64, 2, PK>, 2);
      return go(k_flash_attention<64, 1, PK>, 1);
    }
    if (kv.head_dim == 128) {
      if (groups(2) >= cu) return go(k_flash_attention<128, 2, PK>, 2);
      return go(k_flash_attention<128, 1, PK>, 1);
    }
    return hipErrorInvalidValue;
  };
  return rm.packed ? pick(std::true_type()) : pick(std::false_type());
}

}  // namespace sapo
