// Small decoders (gfx950): a whole rollout or scoring call with one workgroup per sequence.
//
// The shape-generic kernels run one operation of one layer per launch; on a decoder whose matrices are a few hundred KB
// every one of those launches is a few microseconds of latency around a fraction of a microsecond of work (the tiny
// configuration: 23 launches per decode step, 135 us; here 12 us).  Its rollout call, 8 sequences of 16 + 16 tokens, went
// from 2230 to 209 us, scoring 8 x 256 tokens from 360 to 65 us.  Sequences do not
// depend on each other, so here a workgroup of 8 waves takes one sequence through all layers, positions and steps: the
// activations stay in LDS, a workgroup barrier takes the place of a launch, the weights come out of the L2 again for
// every step.
//   k_small_prefill  the positions of a prompt (rollout) or scored sequence in tiles of 16 rows; keys and values go to
//                    global memory, the last position's residual row to h_last, or (scoring) the LM head, log-sum-exp and
//                    target gather of the masked rows follow in the same tile.  Up to kFusedTiles tiles: one workgroup per
//                    sequence and one launch; more: one workgroup per tile and n_layers + 1 launches (tiny decoder,
//                    scoring: two tiles 77 us in one launch, 51 us in three).
//   k_small_decode   one workgroup per sequence: LM head, sampler, embedding and layers of one position, step after step.
// Offsets are 32-bit: small_rows_fit (host; the limits are in ranges.h) says for which calls they are enough.
// What bounds them: a workgroup takes its weights in at 32 bytes a cycle (layers of the tiny decoder: 11.5 of a step's 27
// thousand cycles), and a phase is a chain of dependent instructions between barriers, five per layer.  small_eligible
// (api.hip) says for which models that is still cheaper than the launches.  Per step of the tiny decoder, thousands of
// cycles, before and now: attention 6.3 -> 4.0 a layer (its keys, values and the norms' gains in LDS), other phases of a layer
// 10.2 -> 6.2 (a first pass outside the loop does not wait for the next phase's weights; sums scattered over the lanes, one
// lane's epilogue per feature), LM head 5.1 -> 2.4 (in LDS), sampler 4.4 -> 3.5 (outputs written during the next attention);
// about a third of it all because LDS areas start at multiples of 16 bytes now.
//
// Decode (one row): a product is spread over groups of 16 lanes (lane i takes the k = 4 i .. 4 i + 3 of every 64);
// groups take output features round-robin, so a group's weight request is 256 contiguous bytes and a wave's the rows of
// four features.  The 16 lanes' partial sums meet through DPP lane permutes (no LDS).
// Prefill (16 rows): fp32 matrix cores, 16 features x 16 rows per wave and pass; both operands are read as four
// consecutive k per lane, one per v_mfma_f32_16x16x4_f32 (any assignment of k to slots does, if both operands share it).
// On the vector ALUs the rows' values, read from LDS once per feature, took 2 to 3 times as long.
#include "common.h"
#include "ranges.h"
#include "small.h"
#include <type_traits>

namespace sapo {
namespace {

constexpr int kFusedTiles = 1;
constexpr int kRows = 16;   // rows of a prefill tile: one per lane of a group after the reduction

template <int CTRL> __device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ int dppi(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true); }
// lane controls inside a row of 16: reversed row (i <-> 15 - i), reversed half (i <-> 7 - i), i ^ 2, i ^ 1.  A value
// combined over the four in turn is combined over all 16 lanes.
constexpr int kRor4 = 0x124, kRor8 = 0x128;   // rotated by 4 / 8 inside the row of 16
constexpr int kMirror = 0x140, kHalfMirror = 0x141, kXor2 = 0x4e, kXor1 = 0xb1;

__device__ __forceinline__ float sum16(float x) {
  x += dpp<kMirror>(x); x += dpp<kHalfMirror>(x); x += dpp<kXor2>(x); x += dpp<kXor1>(x);
  return x;
}
__device__ __forceinline__ float wave_sum(float x) { return sum_xor32(sum_xor16(sum16(x))); }
__device__ __forceinline__ float max16(float x) {
  x = fmaxf(x, dpp<kMirror>(x)); x = fmaxf(x, dpp<kHalfMirror>(x)); x = fmaxf(x, dpp<kXor2>(x)); x = fmaxf(x, dpp<kXor1>(x));
  return x;
}
__device__ __forceinline__ float wave_max(float x) { return max_xor32(max_xor16(max16(x))); }
struct Lse { float m, l; };
__device__ __forceinline__ Lse lse_merge(Lse a, Lse b) {
  const float mn = fmaxf(a.m, b.m);
  if (mn == -INFINITY) return a;
  return Lse{mn, a.l * __expf(a.m - mn) + b.l * __expf(b.m - mn)};
}
__device__ __forceinline__ void swap16(float x, float& lo, float& hi) {
  const lane_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo = __uint_as_float(r[0]); hi = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float x, float& lo, float& hi) {
  const lane_u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo = __uint_as_float(r[0]); hi = __uint_as_float(r[1]);
}
__device__ __forceinline__ Lse lse_wave16(Lse a) {   // over the lanes l, l ^ 16, l ^ 32, l ^ 48
  Lse p, q;
  swap16(a.m, p.m, q.m); swap16(a.l, p.l, q.l);
  a = lse_merge(p, q);
  swap32(a.m, p.m, q.m); swap32(a.l, p.l, q.l);
  return lse_merge(p, q);
}
__device__ __forceinline__ BestAcc best_half_row(BestAcc b) {   // over the 8 lanes of a half row
  b.add(dpp<kHalfMirror>(b.y), dpp<kHalfMirror>(b.z), dppi<kHalfMirror>(b.id));
  b.add(dpp<kXor2>(b.y), dpp<kXor2>(b.z), dppi<kXor2>(b.id));
  b.add(dpp<kXor1>(b.y), dpp<kXor1>(b.z), dppi<kXor1>(b.id));
  return b;
}
__device__ __forceinline__ BestAcc best_wave(BestAcc b) {
  b.add(dpp<kMirror>(b.y), dpp<kMirror>(b.z), dppi<kMirror>(b.id));
  b = best_half_row(b);
  float y0, y1, z0, z1, i0, i1;
  swap16(b.y, y0, y1); swap16(b.z, z0, z1); swap16(__int_as_float(b.id), i0, i1);
  b.y = y0; b.z = z0; b.id = __float_as_int(i0);
  b.add(y1, z1, __float_as_int(i1));
  swap32(b.y, y0, y1); swap32(b.z, z0, z1); swap32(__int_as_float(b.id), i0, i1);
  b.y = y0; b.z = z0; b.id = __float_as_int(i0);
  b.add(y1, z1, __float_as_int(i1));
  return b;
}

// Pointers that come out of the layer table are known to the compiler as generic ones: accesses through them become flat
// instructions, which count as LDS operations as well, so that every LDS read would wait for weights requested ahead.
// These say where they point.
template <typename T> using gptr = const T __attribute__((address_space(1)))*;
template <typename T> using gptr_mut = T __attribute__((address_space(1)))*;
template <typename T> __device__ __forceinline__ gptr<T> global(const void* p) { return (gptr<T>)(uintptr_t)p; }
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// four consecutive elements as they are stored (a request, not yet a value)
template <typename T> struct Quad;
template <> struct Quad<float> {
  f32x4 u;
  __device__ __forceinline__ void load(gptr<float> p) { u = *(gptr<f32x4>)p; }
  __device__ __forceinline__ void load(const float* lds) { u = *(const f32x4*)lds; }
  __device__ __forceinline__ float4 f() const { return make_float4(u[0], u[1], u[2], u[3]); }
};
template <> struct Quad<bf16> {
  u32x2 u;
  __device__ __forceinline__ void load(gptr<bf16> p) { u = *(gptr<u32x2>)p; }
  __device__ __forceinline__ void load(const bf16* lds) { u = *(const u32x2*)lds; }
  __device__ __forceinline__ float4 f() const {
    return make_float4(__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16),
                       __uint_as_float(u[1] & 0xffff0000u));
  }
};
__device__ __forceinline__ float4 load4(gptr<float> p) { Quad<float> q; q.load(p); return q.f(); }
template <typename T> __device__ __forceinline__ float rounded(float x) { return to_f32(from_f32<T>(x)); }
__device__ __forceinline__ float fma4(float4 w, float4 x, float acc) {
  return fmaf(w.w, x.w, fmaf(w.z, x.z, fmaf(w.y, x.y, fmaf(w.x, x.x, acc))));
}

constexpr int kThreads = 512, kWaves = kThreads / 64, kGroups = kThreads / 16;
// The thread's index as a value the compiler takes as new each time: nothing derived from it (offsets of every phase)
// is then hoisted out of the loop over the steps and kept in registers across all other phases.
__device__ __forceinline__ int fresh_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
// Features of a pass: group g's feature j is first_feature(n0, j, N) + g, n0 the pass's first.  The last groups of features
// that N does not fill begin early, so that no request needs a bound of its own; what is computed twice is kept once
// (own_feature).  N below kGroups: groups past the end repeat the last feature.
__device__ __forceinline__ int first_feature(int n0, int j, int N) { return max(0, min(n0 + j * kGroups, N - kGroups)); }
__device__ __forceinline__ bool own_feature(int n0, int j, int N, int g) { return g < N && first_feature(n0, j, N) + g >= n0 + j * kGroups; }
// Sums of NF (2, 4, 8, 16) values over the 16 lanes of a group, in the order of sum16; a lane gets value scatter_index (the
// lane's highest bits, the highest first)
template <int NF> __device__ __forceinline__ int scatter_index(int ln) { return ln / (16 / NF); }
template <int NF> __device__ __forceinline__ bool scatter_writer(int ln) { return (ln & (16 / NF - 1)) == 0; }   // one lane per value
template <int NF> __device__ __forceinline__ float scatter16(const float (&in)[NF], int ln) {
  static_assert(NF == 2 || NF == 4 || NF == 8 || NF == 16, "halves");
  float a[16];
#pragma unroll
  for (int i = 0; i < NF; ++i) a[i] = in[i];
  auto step = [&](auto ctrl_c, auto n_c, int bit) __attribute__((always_inline)) {
    constexpr int ctrl = decltype(ctrl_c)::value, n = decltype(n_c)::value;
    if constexpr (n >= 2) {
#pragma unroll
      for (int i = 0; i < n / 2; ++i) a[i] = (ln & bit ? a[i + n / 2] : a[i]) + dpp<ctrl>(ln & bit ? a[i] : a[i + n / 2]);
    } else {
      a[0] += dpp<ctrl>(a[0]);
    }
  };
  step(std::integral_constant<int, kMirror>(), std::integral_constant<int, NF>(), 8);
  step(std::integral_constant<int, kHalfMirror>(), std::integral_constant<int, NF / 2>(), 4);
  step(std::integral_constant<int, kXor2>(), std::integral_constant<int, NF / 4>(), 2);
  step(std::integral_constant<int, kXor1>(), std::integral_constant<int, NF / 8>(), 1);
  return a[0];
}
// The weights of a group's features of one pass, KC chunks of 64 k: requested a phase ahead of their use, since they
// depend on nothing the step computes.
template <typename T, int NF, int KC> struct WeightAhead {
  Quad<T> w[KC][NF];
  template <class P> __device__ __forceinline__ void request(P W, int N, int K, int n0 = 0) {   // P: where W lies, global memory or LDS
    const int ft = fresh_thread(), g = ft >> 4, ln = ft & 15;
    const unsigned row = (unsigned)min(g, N - 1) * K;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const int k = c * 64 + ln * 4;
      const unsigned at = row + (k < K ? k : 0);
#pragma unroll
      for (int j = 0; j < NF; ++j) w[c][j].load(W + (unsigned)first_feature(n0, j, N) * K + at);
    }
  }
};
// y[n] = sum_k W[n][k] x[k] for one row; x(k) gives x[k .. k + 3]; out(n, y) runs in one lane per feature.  NF
// features per group and pass, so that many weight requests are in flight; the first pass takes what `ahead` holds.  It
// stands in front of the loop: in a loop that also requests, the compiler has every use wait for whatever was requested
// last - the next phase's weights, a memory round trip in each phase.
template <typename T, int NF, int KC, class P, class X, class Out>
__device__ __forceinline__ void row_product(const WeightAhead<T, NF, KC>& ahead, P W, int N, int K, X x, Out out) {
  const int ft = fresh_thread(), g = ft >> 4, ln = ft & 15;
  const unsigned row = (unsigned)min(g, N - 1) * K;
  auto rest_of_k = [&](float (&acc)[NF], int n0, int k_first) __attribute__((always_inline)) {
#pragma unroll 1
    for (int k = k_first + ln * 4; k < K; k += 64) {
      Quad<T> w[NF];
#pragma unroll
      for (int j = 0; j < NF; ++j) w[j].load(W + (unsigned)first_feature(n0, j, N) * K + row + k);
      const float4 xv = x(k);
#pragma unroll
      for (int j = 0; j < NF; ++j) acc[j] = fma4(w[j].f(), xv, acc[j]);
    }
  };
  auto emit = [&](const float (&acc)[NF], int n0) __attribute__((always_inline)) {
    const float y = scatter16<NF>(acc, ln);
    const int j = scatter_index<NF>(ln);
    if (scatter_writer<NF>(ln) && own_feature(n0, j, N, g)) out(first_feature(n0, j, N) + g, y);
  };
  float acc[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j) acc[j] = 0.f;
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const int k = c * 64 + ln * 4;
    if (k < K) {
      const float4 xv = x(k);
#pragma unroll
      for (int j = 0; j < NF; ++j) acc[j] = fma4(ahead.w[c][j].f(), xv, acc[j]);
    }
  }
  if (K > KC * 64) rest_of_k(acc, 0, KC * 64);
  emit(acc, 0);
#pragma unroll 1
  for (int n0 = kGroups * NF; n0 < N; n0 += kGroups * NF) {
    float more[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) more[j] = 0.f;
    rest_of_k(more, n0, 0);
    emit(more, n0);
  }
}

// act[n] = silu(gate_n . x) * (up_n . x): gate and up rows of a feature by the same group (W: F gate rows, then F up rows)
template <typename T, int NF, class X>
__device__ __forceinline__ void gate_up(const WeightAhead<T, NF, 1>& ag, const WeightAhead<T, NF, 1>& au, gptr<T> W,
                                        int F, int K, X x, float* act) {
  const int ft = fresh_thread(), g = ft >> 4, ln = ft & 15;
  const gptr<T> Wu = W + (unsigned)F * K;
  const unsigned row = (unsigned)min(g, F - 1) * K;
  auto rest_of_k = [&](float (&yg)[8], float (&yu)[8], int n0, int k_first) __attribute__((always_inline)) {
#pragma unroll 1
    for (int k = k_first + ln * 4; k < K; k += 64) {
      Quad<T> w0[NF], w1[NF];
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        const unsigned at = (unsigned)first_feature(n0, j, F) * K;
        w0[j].load(W + at + row + k); w1[j].load(Wu + at + row + k);
      }
      const float4 xv = x(k);
#pragma unroll
      for (int j = 0; j < NF; ++j) { yg[j] = fma4(w0[j].f(), xv, yg[j]); yu[j] = fma4(w1[j].f(), xv, yu[j]); }
    }
  };
  auto emit = [&](const float (&yg)[8], const float (&yu)[8], int n0) __attribute__((always_inline)) {
    const float a = scatter16<8>(yg, ln), b = scatter16<8>(yu, ln);
    const int j = scatter_index<8>(ln);
    if (scatter_writer<8>(ln) && j < NF && own_feature(n0, j, F, g)) act[first_feature(n0, j, F) + g] = rounded<T>(a / (1.0f + expf(-a)) * b);
  };
  float yg[8] = {}, yu[8] = {};   // NF of them
  if (ln * 4 < K) {
    const float4 xv = x(ln * 4);
#pragma unroll
    for (int j = 0; j < NF; ++j) { yg[j] = fma4(ag.w[0][j].f(), xv, yg[j]); yu[j] = fma4(au.w[0][j].f(), xv, yu[j]); }
  }
  if (K > 64) rest_of_k(yg, yu, 0, 64);
  emit(yg, yu, 0);
#pragma unroll 1
  for (int n0 = kGroups * NF; n0 < F; n0 += kGroups * NF) {
    float mg[8] = {}, mu[8] = {};
    rest_of_k(mg, mu, n0, 0);
    emit(mg, mu, n0);
  }
}

// 16 features from feature n0 on (clamped to N - 1: what lies past it is not to be used) x 16 rows x_lds[r * stride + k]:
// lane l gets features n0 + 4 (l / 16) + v, v < 4, of row l % 16.
template <typename T>
__device__ __forceinline__ f32x4 tile_dot(gptr<T> W, int n0, int N, int K, const float* x_lds, int stride) {
  const int lane = threadIdx.x & 63, g4 = (lane >> 4) * 4;
  const gptr<T> wr = W + (unsigned)min(n0 + (lane & 15), N - 1) * K;
  const float* xr = x_lds + (lane & 15) * stride;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < K; k0 += 64) {   // 64 k at a time, their requests together; K is a multiple of 4: a lane's four k
    Quad<T> w[4];                        // lie inside or past it as a whole, and past it they contribute zeros
    float4 x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = k0 + 16 * i + g4;
      w[i].load(wr + (k < K ? k : 0));
      x[i] = *(const float4*)(xr + (k < K ? k : 0));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = k0 + 16 * i + g4 < K;
      const float4 a = w[i].f();
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? a.x : 0.f, in ? x[i].x : 0.f, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? a.y : 0.f, in ? x[i].y : 0.f, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? a.z : 0.f, in ? x[i].z : 0.f, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? a.w : 0.f, in ? x[i].w : 0.f, acc, 0, 0, 0);
    }
  }
  return acc;
}
// All N features for the tile's rows, 16 per wave and pass: out(n, y) for row lane % 16.
template <typename T, class Out>
__device__ __forceinline__ void tile_product(gptr<T> W, int N, int K, const float* x_lds, int stride, Out out) {
  const int wave = wave_index(threadIdx.x), f0 = ((threadIdx.x & 63) >> 4) * 4;
  for (int n0 = wave * 16; n0 < N; n0 += kWaves * 16) {
    const f32x4 y = tile_dot<T>(W, n0, N, K, x_lds, stride);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (n0 + f0 + v < N) out(n0 + f0 + v, y[v]);
  }
}

__device__ __forceinline__ float rms_scale(const float* h, int d, float eps) {   // by every wave for itself
  float ss = 0.f;
  for (int i = threadIdx.x & 63; i < d; i += 64) ss += h[i] * h[i];
  ss = wave_sum(ss);
  // 1 / sqrtf(ss / d + eps) by the hardware's approximations, each corrected by its residual: fewer dependent instructions and within
  // 1.96 2^-24 of the exact value, where 1 / sqrtf and the division come within 2.33 2^-24 (all sums of four binades, d of 36 .. 132).
  // 8 x (16 + 16) tokens of the tiny decoder 209 us a call, 218 with those.
  const float n = (float)d, inv = 1.0f / n, q = ss * inv, x = fmaf(fmaf(-n, q, ss), inv, q) + eps, r = __builtin_amdgcn_rsqf(x);
  if (!__builtin_isnormal(x)) return 1.0f / sqrtf(ss / n + eps);   // 0, subnormal, infinite
  return fmaf(0.5f * r, fmaf(-x * r, r, 1.0f), r);
}
// a wave's own LDS stores before its own LDS loads
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Keys and values of one layer: [rows][Hkv][hd] each.  Rows 0 .. P Lp - 1 belong to the prompts, then N rows per
// sequence.
template <typename T> __device__ __forceinline__ gptr_mut<T> kv_base(const SmallModel& m, int layer, int which) {
  return (gptr_mut<T>)(uintptr_t)((char*)m.pool + m.pool_bytes * (2 * layer + which));
}
// A layer's pointers through the scalar cache (the table is written when the handle is created)
struct LayerPtrs { const void *wqkv, *wo, *wgu, *wdown; gptr<float> attn_norm, ffn_norm, bqkv; };
__device__ __forceinline__ LayerPtrs layer_ptrs(const SmallModel& m, int l) {
  const SmallLayer __attribute__((address_space(4)))* t = (const SmallLayer __attribute__((address_space(4)))*)(uintptr_t)(m.layers + l);
  return LayerPtrs{t->wqkv, t->wo, t->wgu, t->wdown, global<float>(t->attn_norm), global<float>(t->ffn_norm), global<float>(t->bqkv)};
}

// Softmax attention of one query head by one wave: qs (LDS, rotated, hd
// values) against the rows row(n), n < ctx, of the cache; when `knew` is not null, row ctx - 1 is not in memory yet: its
// key is knew[] and its value vnew[] (LDS).  sc: LDS, ctx floats of the wave.  out[] (LDS) <- the head's output rounded to T.
template <typename T, class Row>
__device__ __forceinline__ void head_attention(const SmallModel& m, gptr<T> kb, gptr<T> vb, int kvh,
                                               int ctx, Row row, const float* qs, const float* knew, const float* vnew, float* sc,
                                               float* out) {
  const int lane = threadIdx.x & 63, hd = m.hd;
  const unsigned rs = (unsigned)m.hkv * hd;
  const float scale = 1.0f / sqrtf((float)hd);
  const int n_mem = knew ? ctx - 1 : ctx;
  // values: a lane takes four dims of every parts-th position; hd / 4 lanes (rounded up to a power of two) cover a
  // position.  The first kAheadV of a lane are requested before the scores.
  constexpr int kAheadV = 8;
  const int quads = hd >> 2;
  int qp = 1;
  while (qp < quads && qp < 64) qp <<= 1;
  const int parts = 64 / qp, part = lane / qp;
  const gptr<T> vq0 = vb + (unsigned)kvh * hd;
  Quad<T> va[kAheadV];
#pragma unroll
  for (int j = 0; j < kAheadV; ++j) {
    const int n = part + j * parts;
    va[j].load(vq0 + 4 * min(lane & (qp - 1), quads - 1) + (unsigned)row(n < n_mem ? n : 0) * rs);
  }
  float mx = -INFINITY;
  for (int n = lane; n < ctx; n += 64) {
    float acc = 0.f;
    if (n < n_mem) {
      const gptr<T> kp = kb + (unsigned)row(n) * rs + (unsigned)kvh * hd;
#pragma unroll 4
      for (int i = 0; i < hd; i += 4) {
        Quad<T> q; q.load(kp + i);
        acc = fma4(q.f(), *(const float4*)(qs + i), acc);
      }
    } else {
      for (int i = 0; i < hd; i += 4) acc = fma4(*(const float4*)(knew + i), *(const float4*)(qs + i), acc);
    }
    acc *= scale;
    sc[n] = acc;
    mx = fmaxf(mx, acc);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int n = lane; n < ctx; n += 64) {
    const float p = expf(sc[n] - mx);
    sc[n] = p;
    sum += p;
  }
  sum = wave_sum(sum);
  wave_sync();
  const float inv = 1.0f / sum;
  for (int iq = lane & (qp - 1); iq < quads; iq += qp) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](const Quad<T>& v, int n) {
      const float4 f = v.f();
      const float p = sc[n];
      acc.x = fmaf(p, f.x, acc.x); acc.y = fmaf(p, f.y, acc.y); acc.z = fmaf(p, f.z, acc.z); acc.w = fmaf(p, f.w, acc.w);
    };
    int n = part;
    if (iq < qp) {
#pragma unroll
      for (int j = 0; j < kAheadV; ++j)
        if (part + j * parts < n_mem) add(va[j], part + j * parts);
      n += kAheadV * parts;
    }
#pragma unroll 8
    for (; n < n_mem; n += parts) {
      Quad<T> v; v.load(vq0 + 4 * iq + (unsigned)row(n) * rs);
      add(v, n);
    }
    if (knew && part == 0) {   // the new position's value, as the cache holds it
      const float p = sc[ctx - 1];
      acc.x = fmaf(p, rounded<T>(vnew[4 * iq]), acc.x); acc.y = fmaf(p, rounded<T>(vnew[4 * iq + 1]), acc.y);
      acc.z = fmaf(p, rounded<T>(vnew[4 * iq + 2]), acc.z); acc.w = fmaf(p, rounded<T>(vnew[4 * iq + 3]), acc.w);
    }
    auto over_parts = [&](float x) {
      if (qp <= 4) {
        if (qp == 1) { x += dpp<kXor1>(x); x += dpp<kXor2>(x); }
        if (qp == 2) x += dpp<kXor2>(x);
        x += dpp<kRor4>(x);
      }
      if (qp <= 8) x += dpp<kRor8>(x);
      if (qp <= 16) x = sum_xor16(x);
      if (qp <= 32) x = sum_xor32(x);
      return x;
    };
    acc.x = over_parts(acc.x); acc.y = over_parts(acc.y); acc.z = over_parts(acc.z); acc.w = over_parts(acc.w);
    if (part == 0)
      *(float4*)(out + 4 * iq) = make_float4(rounded<T>(acc.x * inv), rounded<T>(acc.y * inv), rounded<T>(acc.z * inv), rounded<T>(acc.w * inv));
  }
}

// The same with the sequence's keys and values in LDS (rows k + n stride, v + n stride; position ctx - 1: kn, vn), head dims
// 16, 32, 64; the same sums in the same order.
template <typename T, int HD>
__device__ __forceinline__ void lds_attention(const T* k, const T* v, int stride, int ctx, const float* qs, const T* kn, const T* vn,
                                              float* sc, float* out) {
  constexpr int QP = HD / 4, PARTS = 64 / QP;   // lanes per position; positions of a step
  const int lane = fresh_thread() & 63, iq = lane % QP, part = lane / QP;
  const float scale = 1.0f / sqrtf((float)HD);
  auto quad = [](const T* p) { Quad<T> q; q.load(p); return q.f(); };
  float mx = -INFINITY;
  for (int n = lane; n < ctx; n += 64) {
    const T* kp = n < ctx - 1 ? k + n * stride : kn;
    float acc = 0.f;
#pragma unroll 4
    for (int i = 0; i < HD; i += 4) acc = fma4(quad(kp + i), *(const float4*)(qs + i), acc);
    acc *= scale;
    sc[n] = acc;
    mx = fmaxf(mx, acc);
  }
  mx = wave_max(mx);
  float sum = 0.f;
  for (int n = lane; n < ctx; n += 64) {
    const float p = expf(sc[n] - mx);
    sc[n] = p;
    sum += p;
  }
  sum = wave_sum(sum);
  wave_sync();
  const float inv = 1.0f / sum;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](const T* vp, int n) {
    const float4 f = quad(vp + 4 * iq);
    const float p = sc[n];
    acc.x = fmaf(p, f.x, acc.x); acc.y = fmaf(p, f.y, acc.y); acc.z = fmaf(p, f.z, acc.z); acc.w = fmaf(p, f.w, acc.w);
  };
#pragma unroll 4
  for (int n = part; n < ctx - 1; n += PARTS) add(v + n * stride, n);
  if (part == 0) add(vn, ctx - 1);
  auto over_parts = [](float x) {
    if constexpr (QP <= 4) x += dpp<kRor4>(x);
    if constexpr (QP <= 8) x += dpp<kRor8>(x);
    return sum_xor32(sum_xor16(x));
  };
  acc.x = over_parts(acc.x); acc.y = over_parts(acc.y); acc.z = over_parts(acc.z); acc.w = over_parts(acc.w);
  if (part == 0)
    *(float4*)(out + 4 * iq) = make_float4(rounded<T>(acc.x * inv), rounded<T>(acc.y * inv), rounded<T>(acc.z * inv), rounded<T>(acc.w * inv));
}

// Causal attention of the 16 rows of a tile (positions t0 .. t0 + 15) for one query head by one wave, head dim 16 KK, on
// the fp32 matrix cores: 16 positions at a time, S^T = K Q^T (positions x rows, so that a lane owns one row's statistics),
// online softmax, O^T = V^T P^T with the lane's own probabilities as operand.  Positions past the tile's last row are
// read as that row and masked.
template <typename T, int KK>
__device__ __forceinline__ void tile_attention(gptr<T> kb, gptr<T> vb, unsigned rs, int t0, int n_pos,
                                               const float* qs, int q_stride, float* out, int out_stride) {
  const int lane = threadIdx.x & 63, ln = lane & 15, g = lane >> 4;
  const float scale = 1.0f / sqrtf((float)(16 * KK));
  float4 q[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) q[kk] = *(const float4*)(qs + ln * q_stride + kk * 16 + 4 * g);
  float m = -INFINITY, l = 0.f;
  f32x4 o[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) o[kk] = f32x4{0.f, 0.f, 0.f, 0.f};
  Quad<T> kf[KK];
  T vf[KK][4];
  auto request = [&](int c0) {
    const gptr<T> kp = kb + (unsigned)min(c0 + ln, n_pos - 1) * rs;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk].load(kp + kk * 16 + 4 * g);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const gptr<T> vp = vb + (unsigned)min(c0 + 4 * g + j, n_pos - 1) * rs + ln;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) vf[kk][j] = vp[kk * 16];
    }
  };
  request(0);
  for (int c0 = 0; c0 < n_pos; c0 += 16) {
    float4 k[KK];
    float v[KK][4];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      k[kk] = kf[kk].f();
#pragma unroll
      for (int j = 0; j < 4; ++j) v[kk][j] = to_f32(vf[kk][j]);
    }
    if (c0 + 16 < n_pos) request(c0 + 16);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[kk].x, q[kk].x, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[kk].y, q[kk].y, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[kk].z, q[kk].z, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[kk].w, q[kk].w, s, 0, 0, 0);
    }
    float p[4], mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      p[j] = c0 + 4 * g + j <= t0 + ln ? s[j] * scale : -INFINITY;
      mx = fmaxf(mx, p[j]);
    }
    mx = max_xor32(max_xor16(mx));
    const float mn = fmaxf(m, mx), alpha = expf(m - mn);   // position 0 is open to every row: mn is finite
    float ps = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) { p[j] = expf(p[j] - mn); ps += p[j]; }
    l = l * alpha + ps;
    m = mn;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
#pragma unroll
      for (int j = 0; j < 4; ++j) o[kk][j] *= alpha;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[kk] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[kk][j], p[j], o[kk], 0, 0, 0);
    }
  }
  const float inv = 1.0f / sum_xor32(sum_xor16(l));
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    *(float4*)(out + ln * out_stride + kk * 16 + 4 * g) =
        make_float4(rounded<T>(o[kk][0] * inv), rounded<T>(o[kk][1] * inv), rounded<T>(o[kk][2] * inv), rounded<T>(o[kk][3] * inv));
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_small_prefill(SmallModel m, SmallPrefill a) {
  extern __shared__ __align__(16) float smem[];   // behind 8 bytes more than a multiple of 16, every 16-byte access would be split
  const int d = m.d, q = m.hq * m.hd, kvd = m.hkv * m.hd, nq = q + 2 * kvd, F = m.F, half = m.hd / 2;
  const int sa = max(d, q);
  float* h = smem;                      // [16][d]
  float* x = h + kRows * d;             // [16][max(d, q)] norm output, then attention output
  float* u = x + kRows * sa;            // [16][max(nq, F)] q / k / v, then the SwiGLU product
  float* sc = u + kRows * max(nq, F);   // [waves][T] scores
  const int tid = threadIdx.x, wave = wave_index(tid), lane = tid & 63, ln = tid & 15;
  const int s = blockIdx.x;
  const int len = a.lens ? a.lens[s] : a.T;
  const int32_t* tok = a.tokens + (unsigned)s * a.T;
  const unsigned row0 = (unsigned)s * a.T;
  // One launch for everything (stage < 0): this workgroup takes the sequence's tiles one after the other through all
  // layers.  Staged: a workgroup per tile and one launch per stage; stage l ends layer l - 1 (from its attention on) and
  // begins layer l (up to its keys and values), so that a tile finds the keys and values of all tiles before it.
  const bool staged = a.stage >= 0;
  const int t_begin = staged ? (int)blockIdx.y * kRows : 0, t_end = staged ? min(len, t_begin + kRows) : len;
  const int st_begin = staged ? a.stage : 0, st_end = staged ? a.stage : m.L;
  for (int t0 = t_begin; t0 < t_end; t0 += kRows) {
    const int nr = min(kRows, len - t0);
    __syncthreads();   // the tile before is done with LDS
    for (int i = tid; i < kRows * d; i += kThreads) {
      const int r = i / d;
      h[i] = r >= nr ? 0.f : st_begin == 0 ? to_f32(((const T*)m.embed)[(unsigned)tok[t0 + r] * d + (i - r * d)])
                                           : a.h_rows[(row0 + t0) * d + i];
    }
    if (st_begin > 0) {   // the rotated queries the stage before left behind
      for (int i = tid; i < kRows * q; i += kThreads) {
        const int r = i / q;
        u[r * nq + (i - r * q)] = r < nr ? to_f32(((const T*)a.q_rows)[(row0 + t0) * q + i]) : 0.f;
      }
    }
    __syncthreads();
    auto norm = [&](gptr<float> gain) {
      for (int r = wave; r < kRows; r += kWaves) {
        const float sc_r = rms_scale(h + r * d, d, m.eps);
        for (int i = lane; i < d; i += 64) x[r * sa + i] = rounded<T>(h[r * d + i] * sc_r * gain[i]);
      }
      __syncthreads();
    };
    for (int stage = st_begin; stage <= st_end; ++stage) {
      if (stage > 0) {
        const int l = stage - 1;
        const LayerPtrs w = layer_ptrs(m, l);
        const gptr_mut<T> kb = kv_base<T>(m, l, 0), vb = kv_base<T>(m, l, 1);
        if (m.hd == 16 || m.hd == 32 || m.hd == 64) {
          for (int head = wave; head < m.hq; head += kWaves) {
            const unsigned rs = (unsigned)kvd, o = row0 * rs + (unsigned)(head / (m.hq / m.hkv)) * m.hd;
            const float* qs = u + head * m.hd;
            float* out = x + head * m.hd;
            if (m.hd == 16) tile_attention<T, 1>(kb + o, vb + o, rs, t0, t0 + nr, qs, nq, out, sa);
            else if (m.hd == 32) tile_attention<T, 2>(kb + o, vb + o, rs, t0, t0 + nr, qs, nq, out, sa);
            else tile_attention<T, 4>(kb + o, vb + o, rs, t0, t0 + nr, qs, nq, out, sa);
          }
        } else {
          for (int i = wave; i < nr * m.hq; i += kWaves) {
            const int r = i / m.hq, head = i - r * m.hq;
            head_attention<T>(m, kb, vb, head / (m.hq / m.hkv), t0 + r + 1, [&](int n) { return row0 + n; },
                              u + r * nq + head * m.hd, nullptr, nullptr, sc + (unsigned)wave * a.T, x + r * sa + head * m.hd);
            wave_sync();
          }
        }
        __syncthreads();
        tile_product<T>(global<T>(w.wo), d, q, x, sa, [&](int n, float y) { h[ln * d + n] += y; });
        __syncthreads();
        norm(w.ffn_norm);
        for (int n0 = wave * 16; n0 < F; n0 += kWaves * 16) {   // gate and up of a feature in the same lane
          const f32x4 yg = tile_dot<T>(global<T>(w.wgu), n0, F, d, x, sa);
          const f32x4 yu = tile_dot<T>(global<T>(w.wgu) + (unsigned)F * d, n0, F, d, x, sa);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int n = n0 + (lane >> 4) * 4 + v;
            if (n < F) u[ln * F + n] = rounded<T>(yg[v] / (1.0f + expf(-yg[v])) * yu[v]);
          }
        }
        __syncthreads();
        tile_product<T>(global<T>(w.wdown), d, F, u, F, [&](int n, float y) { h[ln * d + n] += y; });
        __syncthreads();
      }
      if (stage < m.L) {
        const LayerPtrs w = layer_ptrs(m, stage);
        const gptr_mut<T> kb = kv_base<T>(m, stage, 0), vb = kv_base<T>(m, stage, 1);
        norm(w.attn_norm);
        tile_product<T>(global<T>(w.wqkv), nq, d, x, sa, [&](int n, float y) { u[ln * nq + n] = w.bqkv ? y + w.bqkv[n] : y; });
        __syncthreads();
        // rotary: queries in place (staged: to memory), keys and values to the cache
        for (int i = tid; i < nr * (nq / 2); i += kThreads) {
          const int r = i / (nq / 2), j = i - r * (nq / 2), head = j / half, e = j - head * half;
          float* p = u + r * nq + head * m.hd + e;
          const float x1 = p[0], x2 = p[half];
          const int hk = head - m.hq;
          const unsigned o = ((row0 + t0 + r) * m.hkv + (unsigned)(hk < m.hkv ? hk : hk - m.hkv)) * m.hd + e;
          if (hk >= m.hkv) {
            vb[o] = from_f32<T>(x1); vb[o + half] = from_f32<T>(x2);
          } else {
            const float2 cs = m.rope[(unsigned)(t0 + r) * half + e];
            const T r1 = from_f32<T>(x1 * cs.x - x2 * cs.y), r2 = from_f32<T>(x2 * cs.x + x1 * cs.y);
            if (hk >= 0) {
              kb[o] = r1; kb[o + half] = r2;
            } else if (staged) {
              T* qo = (T*)a.q_rows + (row0 + t0 + r) * (unsigned)q + head * m.hd + e;
              qo[0] = r1; qo[half] = r2;
            } else {
              p[0] = to_f32(r1); p[half] = to_f32(r2);
            }
          }
        }
        __syncthreads();
      }
    }
    if (st_end < m.L) {
      for (int i = tid; i < nr * d; i += kThreads) a.h_rows[(row0 + t0) * d + i] = h[i];
      continue;
    }
    if (a.h_last) {
      if (t0 + nr == len)
        for (int i = tid; i < d; i += kThreads) a.h_last[(unsigned)s * d + i] = h[(nr - 1) * d + i];
      continue;
    }
    if (a.out_adv && t0 == 0 && s % a.G == 0 && tid == 0) group_advantages(a.rewards + s, a.G, a.out_adv + s);
    if (t0 == 0 && tid == 0) a.out_logprobs[row0] = 0.f;
    // scoring: row r of the tile predicts the token at t0 + r + 1
    const int t = t0 + ln + 1;
    const bool wanted = ln < nr && t < a.T && a.mask[row0 + t] != 0;
    if (tid < nr && t < a.T && !wanted) a.out_logprobs[row0 + t] = 0.f;
    if (!__syncthreads_or(wanted ? 1 : 0)) continue;
    {
      for (int r = wave; r < kRows; r += kWaves) {
        const float sc_r = rms_scale(h + r * d, d, m.eps);
        for (int i = lane; i < d; i += 64) {
          // log softmax(z / T): z is linear in the final norm's gains, so the temperature goes into them
          const float gain = a.inv_t == 1.0f ? m.final_norm[i] : m.final_norm[i] * a.inv_t;
          x[r * sa + i] = rounded<T>(h[r * d + i] * sc_r * gain);
        }
      }
      __syncthreads();
    }
    const int target = wanted ? tok[t] : -1;
    Lse acc{-INFINITY, 0.f};
    tile_product<T>(global<T>(m.lm_head), m.V, d, x, sa, [&](int n, float y) {
      acc = lse_merge(acc, Lse{y, 1.f});
      if (n == target) u[ln] = y;
    });
    acc = lse_wave16(acc);
    float* part = u + 16;   // [waves][16 rows][2]
    if (lane < 16) { part[(wave * 16 + ln) * 2] = acc.m; part[(wave * 16 + ln) * 2 + 1] = acc.l; }
    __syncthreads();
    if (tid < 16 && wanted) {
      Lse z{part[ln * 2], part[ln * 2 + 1]};
      for (int w = 1; w < kWaves; ++w) z = lse_merge(z, Lse{part[(w * 16 + ln) * 2], part[(w * 16 + ln) * 2 + 1]});
      a.out_logprobs[row0 + t] = u[ln] - (z.m + logf(z.l));
    }
  }
}

// RES: the norms' gains and the sequence's keys and values stay in LDS for the whole call (where everything fits and the head
// dim is 16, 32 or 64).  What it is for: read from memory, every phase's gains and keys were requested last and waited for
// first, behind the weights requested ahead.
template <typename T, bool RES>
__global__ void __launch_bounds__(kThreads) k_small_decode(SmallModel m, SmallDecode a) {
  extern __shared__ __align__(16) float smem[];   // behind 8 bytes more than a multiple of 16, every 16-byte access would be split
  const int d = m.d, q = m.hq * m.hd, kvd = m.hkv * m.hd, nq = q + 2 * kvd, F = m.F, half = m.hd / 2, V = m.V;
  float* h = smem;                       // [d]
  float* u = h + d;                      // [max(nq, F)] q / k / v, then the SwiGLU product
  float* at = u + max(nq, F);            // [q] attention output
  constexpr int HW = RES ? 3 : 2;        // vectors of a wave: its rotated query and key (RES: and value)
  float* hw = at + q;                    // [waves][HW hd]
  float* noise = hw + kWaves * HW * m.hd; // [V] the step's Gumbel noise
  const int v4 = RES ? (V + 3) & ~3 : V;
  float* sc = noise + v4;                // [max(V, waves x ctx)] logits, then scores
  // RES: [2 L + 1][d] gains; [L][2][ctx_max] rows of kv_row keys or values, 16 bytes apart from a multiple of the banks
  float* gains = sc + ((max(V, kWaves * a.ctx_max) + 3) & ~3);
  T* kv_lds = (T*)(gains + (2 * m.L + 1) * d);
  const int kv_row = kvd + 16 / (int)sizeof(T);
  T* lm_lds = kv_lds + 2 * m.L * a.ctx_max * kv_row;   // a.lm_resident: [V][d], 16-byte aligned (as every area in front)
  __shared__ float s_m[kWaves], s_l[kWaves], s_y[kWaves], s_z[kWaves];
  __shared__ int s_id[kWaves], s_tok, s_end;
  const int tid = threadIdx.x, wave = wave_index(tid), lane = tid & 63;
  const int s = blockIdx.x, p = s / a.G;
  const int len = a.lens ? a.lens[p] : a.Lp;
  const int rep = m.hq / m.hkv;
  const unsigned own0 = (unsigned)a.P * a.Lp + (unsigned)s * a.N;   // cache row of the sequence's first generated token
  for (int i = tid; i < d; i += kThreads) h[i] = a.h_last[(unsigned)p * d + i];
  if (tid == 0) s_end = 0;
  if constexpr (RES) {
    for (int l = 0; l < m.L; ++l) {
      const LayerPtrs w = layer_ptrs(m, l);
      for (int i = tid; i < d; i += kThreads) {
        gains[2 * l * d + i] = w.attn_norm[i];
        gains[(2 * l + 1) * d + i] = w.ffn_norm[i];
      }
      for (int i = tid; i < len * (kvd / 4); i += kThreads) {
        const int n = i / (kvd / 4), c = 4 * (i - n * (kvd / 4));
        const unsigned o = ((unsigned)p * a.Lp + n) * kvd + c;
#pragma unroll
        for (int which = 0; which < 2; ++which) {
          Quad<T> x;
          x.load((gptr<T>)kv_base<T>(m, l, which) + o);
          *(decltype(x.u)*)(kv_lds + (unsigned)(2 * l + which) * a.ctx_max * kv_row + n * kv_row + c) = x.u;
        }
      }
    }
    for (int i = tid; i < d; i += kThreads) gains[2 * m.L * d + i] = m.final_norm[i];
    if (a.lm_resident) {
#pragma unroll 8
      for (int i = tid; i < V * d / 4; i += kThreads) {
        Quad<T> x;
        x.load(global<T>(m.lm_head) + 4 * (unsigned)i);
        *(decltype(x.u)*)(lm_lds + 4 * i) = x.u;
      }
    }
  }
  __syncthreads();
  // The noise of a step does not depend on the logits: the waves without a query head draw it during the last layer's
  // attention of that step (all waves, if every wave has one).
  const int first_idle = m.hq < kWaves ? m.hq : 0;
  auto draw_noise = [&](int step, int wave0) {
    if (a.temperature == 0.f || wave < wave0) return;
    for (int b = tid - wave0 * 64; b < (V + 3) / 4; b += kThreads - wave0 * 64) {
      float g[4];
      gumbel4(a.seed_lo, a.seed_hi, (uint32_t)s, (uint32_t)step, (uint32_t)b, g);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * b + j < V) noise[4 * b + j] = g[j];
    }
  };
  auto normed = [&](gptr<float> gain, int which, float scl) {   // norm `which`: 2 l, 2 l + 1, 2 L
    return [=](int k) {
      float4 gv;
      if constexpr (RES) gv = *(const float4*)(gains + which * d + k);
      else gv = load4(gain + k);
      const float4 hv = *(const float4*)(h + k);
      return make_float4(rounded<T>(hv.x * scl * gv.x), rounded<T>(hv.y * scl * gv.y), rounded<T>(hv.z * scl * gv.z),
                         rounded<T>(hv.w * scl * gv.w));
    };
  };
  const gptr<T> lm = global<T>(m.lm_head);
  WeightAhead<T, 4, 1> w_qkv;
  w_qkv.request(global<T>(layer_ptrs(m, 0).wqkv), nq, d);
  draw_noise(0, 0);
  static_assert(kWaves == 8, "one wave's result per lane of a half row");
  auto best_of_waves = [&] {
    BestAcc b;
    b.y = s_y[lane & 7]; b.z = s_z[lane & 7]; b.id = s_id[lane & 7];
    return best_half_row(b);
  };
  // The outputs of step `at` from the waves' results, which stand until the next logits: by one wave, while the others are in
  // the next step's first attention.
  auto write_outputs = [&](int at) {
    if (wave != kWaves - 1) return;
    const BestAcc b = best_of_waves();
    Lse lse{s_m[lane & 7], s_l[lane & 7]};
    lse = lse_merge(lse, Lse{dpp<kHalfMirror>(lse.m), dpp<kHalfMirror>(lse.l)});
    lse = lse_merge(lse, Lse{dpp<kXor2>(lse.m), dpp<kXor2>(lse.l)});
    lse = lse_merge(lse, Lse{dpp<kXor1>(lse.m), dpp<kXor1>(lse.l)});
    if (lane == 0) {
      const bool good = (unsigned)b.id < (unsigned)V;
      a.out_tokens[(unsigned)s * a.N + at] = good ? b.id : -1;
      a.out_logprobs[(unsigned)s * a.N + at] = good ? b.z - (lse.m + logf(lse.l)) : 0.f;
    }
  };
  int t = 0;
  for (;;) {
    // ---- the token of step t: logits, log-sum-exp, Gumbel-max
    {
      auto logits = [&](auto W) __attribute__((always_inline)) {
        WeightAhead<T, 16, 1> w_lm;
        w_lm.request(W, V, d);
        row_product<T>(w_lm, W, V, d, normed(global<float>(m.final_norm), 2 * m.L, rms_scale(h, d, m.eps)), [&](int n, float y) { sc[n] = y; });
      };
      if (RES && a.lm_resident) logits((const T*)lm_lds);
      else logits(lm);
      __syncthreads();
      // every wave: the maximum of its logits, then the sum of exponentials around it, and its best perturbed score
      float mx = -INFINITY;
      BestAcc best; best.init();
      for (int v = tid; v < V; v += kThreads) {
        const float zv = sc[v];
        mx = fmaxf(mx, zv);
        best.add(a.temperature != 0.f ? zv / a.temperature + noise[v] : zv, zv, v);
      }
      mx = wave_max(mx);
      float sum = 0.f;
      if (mx > -INFINITY)
        for (int v = tid; v < V; v += kThreads) sum += __expf(sc[v] - mx);
      sum = wave_sum(sum);
      best = best_wave(best);
      if (lane == 0) { s_m[wave] = mx; s_l[wave] = sum; s_y[wave] = best.y; s_z[wave] = best.z; s_id[wave] = best.id; }
      __syncthreads();
      if (wave == 0) {
        best = best_of_waves();
        if (lane == 0) {
          const int tk = (unsigned)best.id < (unsigned)V ? best.id : -1;   // -1: no score beat the initial one: the logits are not numbers
          s_end = a.stop_token >= 0 && tk == a.stop_token;
          s_tok = tk < 0 ? 0 : tk;
        }
      }
      __syncthreads();
    }
    if (s_end || t + 1 == a.N) break;
    for (int i = tid; i < d; i += kThreads) h[i] = to_f32(((const T*)m.embed)[(unsigned)s_tok * d + i]);
    ++t;
    __syncthreads();
    const int pos = len + t - 1, ctx = pos + 1;
    const float2 cs_pos = m.rope[(unsigned)pos * half + min(lane, half - 1)];
    for (int l = 0; l < m.L; ++l) {
      const LayerPtrs w = layer_ptrs(m, l);
      const gptr_mut<T> kb = kv_base<T>(m, l, 0), vb = kv_base<T>(m, l, 1);
      WeightAhead<T, 2, 1> w_o;
      w_o.request(global<T>(w.wo), d, q);
      row_product<T>(w_qkv, global<T>(w.wqkv), nq, d, normed(w.attn_norm, 2 * l, rms_scale(h, d, m.eps)),
                  [&](int n, float y) { u[n] = w.bqkv ? y + w.bqkv[n] : y; });
      __syncthreads();
      if (l == m.L - 1) draw_noise(t, first_idle);
      if (l == 0) write_outputs(t - 1);
      WeightAhead<T, 6, 1> w_g, w_u;
      auto request_gate_up = [&] {
        w_g.request(global<T>(w.wgu), F, d);
        w_u.request(global<T>(w.wgu) + (unsigned)F * d, F, d);
      };
      if constexpr (RES) {
        request_gate_up();   // nothing of the attention waits behind them
        for (int head = wave; head < m.hq; head += kWaves) {
          const int kvh = head / rep;
          float* qs = hw + wave * HW * m.hd;
          T *kn = (T*)(qs + m.hd), *vn = (T*)(qs + 2 * m.hd);
          T *kl = kv_lds + (unsigned)(2 * l) * a.ctx_max * kv_row + kvh * m.hd, *vl = kl + (unsigned)a.ctx_max * kv_row;
          for (int e = fresh_thread() & 63; e < half; e += 64) {
            const float q1 = u[head * m.hd + e], q2 = u[head * m.hd + e + half];
            const float k1 = u[q + kvh * m.hd + e], k2 = u[q + kvh * m.hd + e + half];
            qs[e] = rounded<T>(q1 * cs_pos.x - q2 * cs_pos.y); qs[e + half] = rounded<T>(q2 * cs_pos.x + q1 * cs_pos.y);
            const T r1 = from_f32<T>(k1 * cs_pos.x - k2 * cs_pos.y), r2 = from_f32<T>(k2 * cs_pos.x + k1 * cs_pos.y);
            const T w1 = from_f32<T>(u[q + kvd + kvh * m.hd + e]), w2 = from_f32<T>(u[q + kvd + kvh * m.hd + e + half]);
            kn[e] = r1; kn[e + half] = r2;
            vn[e] = w1; vn[e + half] = w2;
            if (head == kvh * rep) {   // read from the next step on
              kl[pos * kv_row + e] = r1; kl[pos * kv_row + e + half] = r2;
              vl[pos * kv_row + e] = w1; vl[pos * kv_row + e + half] = w2;
            }
          }
          wave_sync();
          float *scw = sc + (unsigned)wave * a.ctx_max, *out = at + head * m.hd;
          if (m.hd == 16) lds_attention<T, 16>(kl, vl, kv_row, ctx, qs, kn, vn, scw, out);
          else if (m.hd == 32) lds_attention<T, 32>(kl, vl, kv_row, ctx, qs, kn, vn, scw, out);
          else lds_attention<T, 64>(kl, vl, kv_row, ctx, qs, kn, vn, scw, out);
          wave_sync();
        }
        __syncthreads();
      } else {
      // a wave per query head: it rotates its query and, for itself, the new key
      for (int head = wave; head < m.hq; head += kWaves) {
        const int kvh = head / rep;
        float* qs = hw + wave * HW * m.hd;
        float* kn = qs + m.hd;
        float* vn = u + q + kvd + kvh * m.hd;
        for (int e = lane; e < half; e += 64) {
          const float2 cs = e < 64 ? cs_pos : m.rope[(unsigned)pos * half + e];
          const float q1 = u[head * m.hd + e], q2 = u[head * m.hd + e + half];
          const float k1 = u[q + kvh * m.hd + e], k2 = u[q + kvh * m.hd + e + half];
          qs[e] = rounded<T>(q1 * cs.x - q2 * cs.y); qs[e + half] = rounded<T>(q2 * cs.x + q1 * cs.y);
          const T r1 = from_f32<T>(k1 * cs.x - k2 * cs.y), r2 = from_f32<T>(k2 * cs.x + k1 * cs.y);
          kn[e] = to_f32(r1); kn[e + half] = to_f32(r2);
          if (head == kvh * rep) {
            const unsigned o = ((own0 + t - 1) * m.hkv + kvh) * m.hd + e;
            kb[o] = r1; kb[o + half] = r2;
            vb[o] = from_f32<T>(vn[e]); vb[o + half] = from_f32<T>(vn[e + half]);
          }
        }
        wave_sync();
        head_attention<T>(m, kb, vb, kvh, ctx, [&](int n) { return n < len ? (unsigned)p * a.Lp + n : own0 + (n - len); }, qs, kn,
                          vn, sc + (unsigned)wave * a.ctx_max, at + head * m.hd);
        wave_sync();
      }
      request_gate_up();
      __syncthreads();
      }
      row_product<T>(w_o, global<T>(w.wo), d, q, [&](int k) { return *(const float4*)(at + k); }, [&](int n, float y) {
        h[n] += y;
      });
      WeightAhead<T, 2, 3> w_d;
      w_d.request(global<T>(w.wdown), d, F);
      __syncthreads();
      {
        // a group's gate and up features side by side: the product is taken in the lane
        const auto x = normed(w.ffn_norm, 2 * l + 1, rms_scale(h, d, m.eps));
        gate_up<T>(w_g, w_u, global<T>(w.wgu), F, d, x, u);
      }
      w_qkv.request(global<T>(layer_ptrs(m, l + 1 < m.L ? l + 1 : 0).wqkv), nq, d);   // after the last layer: the next step's first
      __syncthreads();
      row_product<T>(w_d, global<T>(w.wdown), d, F, [&](int k) { return *(const float4*)(u + k); }, [&](int n, float y) {
        h[n] += y;
      });
      __syncthreads();
    }
  }
  write_outputs(t);
  // an ended sequence's row goes on as padding
  for (int i = t + 1 + tid; i < a.N; i += kThreads) {
    a.out_tokens[(unsigned)s * a.N + i] = a.stop_token;
    a.out_logprobs[(unsigned)s * a.N + i] = 0.f;
  }
  if (tid == 0 && a.out_lengths) a.out_lengths[s] = t + 1;
}

size_t prefill_lds(const SmallModel& m, int T) {
  const size_t d = m.d, q = (size_t)m.hq * m.hd, nq = q + 2 * (size_t)m.hkv * m.hd, F = m.F;
  size_t u = kRows * (nq > F ? nq : F);
  if (u < 16 + kWaves * 32) u = 16 + kWaves * 32;
  return (kRows * d + kRows * (d > q ? d : q) + u + (size_t)kWaves * T) * sizeof(float);
}
size_t decode_lds(const SmallModel& m, int ctx_max, bool res, size_t elt) {
  const size_t d = m.d, q = (size_t)m.hq * m.hd, kvd = (size_t)m.hkv * m.hd, nq = q + 2 * kvd, F = m.F, V = m.V;
  const size_t sc = (size_t)kWaves * ctx_max;
  if (!res) return (d + (nq > F ? nq : F) + q + kWaves * 2 * (size_t)m.hd + V + (V > sc ? V : sc)) * sizeof(float);
  const auto four = [](size_t n) { return (n + 3) & ~(size_t)3; };
  return (d + (nq > F ? nq : F) + q + kWaves * 3 * (size_t)m.hd + four(V) + four(V > sc ? V : sc) + (2 * (size_t)m.L + 1) * d) * sizeof(float) +
         2 * (size_t)m.L * ctx_max * (kvd * elt + 16);
}
constexpr size_t kLdsLimit = 150 * 1024;
constexpr size_t kDecodeLds = 159 * 1024;   // a workgroup has its compute unit to itself

template <typename T> hipError_t set_lds() {
  hipError_t e = hipFuncSetAttribute((const void*)k_small_prefill<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)k_small_decode<T, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDecodeLds);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_small_decode<T, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
}
hipError_t set_lds_once(int dtype) {
  static bool done[2] = {false, false};
  if (done[dtype == SAPO_DTYPE_BF16]) return hipSuccess;
  const hipError_t e = dtype == SAPO_DTYPE_BF16 ? set_lds<bf16>() : set_lds<float>();
  if (e == hipSuccess) done[dtype == SAPO_DTYPE_BF16] = true;
  return e;
}

}  // namespace

// positions in the cache of a call, prompt (or scored) positions, elements of its largest int32 / fp32 input or output
bool small_rows_fit(const SmallModel& m, size_t cache_rows, size_t prompt_rows, size_t io_elems) {
  return small_offsets_fit(m.d, (uint64_t)m.hq * m.hd, (uint64_t)m.hkv * m.hd, cache_rows, prompt_rows, io_elems);
}
bool small_prefill_fits(const SmallModel& m, int T) { return prefill_lds(m, T) <= kLdsLimit; }
bool small_decode_fits(const SmallModel& m, int ctx_max) { return decode_lds(m, ctx_max, false, 4) <= kLdsLimit; }

hipError_t small_prefill(int dtype, const SmallModel& m, const SmallPrefill& args, int n_seq, hipStream_t st) {
  if (n_seq <= 0 || args.T <= 0 || !small_prefill_fits(m, args.T)) return hipErrorInvalidValue;
  hipError_t e = set_lds_once(dtype);
  if (e != hipSuccess) return e;
  const size_t lds = prefill_lds(m, args.T);
  const int tiles = (args.T + kRows - 1) / kRows;
  const bool fused = tiles <= kFusedTiles;
  SmallPrefill a = args;
  for (int stage = fused ? -1 : 0; stage <= (fused ? -1 : m.L); ++stage) {
    a.stage = stage;
    const dim3 grid(n_seq, fused ? 1 : tiles);
    if (dtype == SAPO_DTYPE_F32) e = launch(KID_SMALL, k_small_prefill<float>, grid, dim3(kThreads), lds, st, m, a);
    else e = launch(KID_SMALL, k_small_prefill<bf16>, grid, dim3(kThreads), lds, st, m, a);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t small_decode(int dtype, const SmallModel& m, const SmallDecode& args, int S, hipStream_t st) {
  if (S <= 0 || !small_decode_fits(m, args.ctx_max)) return hipErrorInvalidValue;
  SmallDecode a = args;
  const hipError_t e = set_lds_once(dtype);
  if (e != hipSuccess) return e;
  const size_t elt = dtype == SAPO_DTYPE_F32 ? 4 : 2;
  // One token per sequence: no step's attention follows and the head is read once, so nothing is worth a copy into LDS.  us a call of
  // the tiny decoder with the copies and without, 64 x 8 sequences of 16 + 1 tokens 49.7, 44.8;
  // 128 + 1 112, 101; with two tokens they pay (16 + 2 72, before there were any 81).
  const bool res = a.N > 1 && (m.hd == 16 || m.hd == 32 || m.hd == 64) && decode_lds(m, a.ctx_max, true, elt) <= kDecodeLds;
  size_t lds = decode_lds(m, a.ctx_max, res, elt);
  const size_t head = (size_t)m.V * m.d * elt;   // the LM head too, where it fits behind the rest
  a.lm_resident = res && head <= kDecodeLds - lds;
  if (a.lm_resident) lds += head;
  auto go = [&](auto kernel) { return launch(KID_SMALL, kernel, dim3(S), dim3(kThreads), lds, st, m, a); };
  if (dtype == SAPO_DTYPE_F32) return res ? go(k_small_decode<float, true>) : go(k_small_decode<float, false>);
  return res ? go(k_small_decode<bf16, true>) : go(k_small_decode<bf16, false>);
}

}  // namespace sapo
