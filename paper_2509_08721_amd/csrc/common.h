// Internal declarations shared by the translation units of libsapo (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <tuple>
#include <stddef.h>

#include "../../include/sapo.h"

namespace sapo {

typedef __bf16 bf16;
typedef _Float16 f16;   // MFMA operand type: packed weights, activations, KV cache of the MFMA path

constexpr int kPageTokens = 16;
constexpr int kWave = 64;

// ---------------------------------------------------------------------------------------
// Row -> (sequence, position) maps.  A "row" is one token being pushed through the layers.
//   block mode : rows are laid out [n_seq, T]; row m is position m % T of cache sequence
//                (m / T) * seq_stride (prefill of prompt p writes through the page table of
//                the first sibling, seq_stride = G; scoring uses seq_stride = 1).
//   decode mode: row m is sequence m at position Lp + *step - 1 (the token sampled at the
//                previous step); *step lives in device memory so that one captured graph
//                can be replayed for every step.
// Prompts of different lengths (optional): lens[p] is the length of prompt p = sequence / G.  Block rows
// at or past their prompt's length are padding: they run through the layers but leave no K/V behind;
// decode rows sit at lens[p] + *step - 1.
// ---------------------------------------------------------------------------------------
struct RowMap {
  int decode;       // 0 block, 1 decode
  int T;            // block mode: positions per sequence
  int seq_stride;   // block mode: cache-sequence stride
  int Lp;           // decode mode: prompt length
  const int* step;  // decode mode: device pointer to the current step index (>= 1)
  const int* lens;  // optional, device: prompt lengths
  int G;            // sequences per prompt (with lens)
  // decode mode, optional, device: the sequence behind each row once ended sequences have been taken out of
  // the batch (row m of the step's activations belongs to sequence slot_seq[m]); NULL: row m is sequence m
  const int* slot_seq = nullptr;
  // block mode, optional, device (g_packed_rows): only the positions that a result depends on, side by side.  Row m lies on page
  // packed[m].x of the cache at position packed[m].y of its sequence; sequence s begins at row first[s], and first[number of
  // sequences] is how many rows there are.  NULL: every sequence has T rows
  const int2* packed = nullptr;
  const int* first = nullptr;
  __device__ __forceinline__ void get(int m, int& seq, int& pos) const {
    if (decode) {
      seq = slot_seq ? slot_seq[m] : m;
      pos = (lens ? lens[seq / G] : Lp) + *step - 1;
    } else {
      seq = (m / T) * seq_stride;
      pos = m % T;
    }
  }
  // does row m leave K/V in the cache?
  __device__ __forceinline__ bool keeps_kv(int m) const { return decode || packed || !lens || (m % T) < lens[m / T]; }
};

// Paged KV cache of one layer.  K and V page: [Hkv] x 16 tokens of hd values, for the shape-generic kernels K as
// [16 tokens][hd] and V as [hd][16 tokens] (token-minor: a fixed feature's 16 tokens are contiguous).
// Element type: fp32 for fp32 models; for bf16 models the shape-generic kernels keep bf16 and the
// MFMA kernels keep IEEE half (same 2 bytes, 3 more mantissa bits: attention involves no weights,
// so its operands need not share the weights' type; values are clamped to the half range).
// Inside a page and head the MFMA kernels keep the order in which a wave reads it as operands (k_page_at, v_page_at).
struct KVCache {
  void* k;                // [n_pages][Hkv] pages
  void* v;                // [n_pages][Hkv] pages
  const int* page_table;  // [n_cache_seq][pages_per_seq]
  int pages_per_seq;
  int n_kv_heads;
  int head_dim;
};

// Element order of a page of one head on the MFMA path.  A wave reads two pages (32 tokens) as K fragments (t, kk) - lane l:
// token 8 ((l % 16) / 4) + 4 t + l % 4, dims 32 kk + 8 (l / 16) .. + 7 - and V fragments dt - lane l: dim 16 dt + l % 16, tokens
// 8 (l / 16) .. + 7 - 16 bytes per lane.  Both are laid out so that eight (K) or sixteen (V) neighbouring lanes read
// neighbouring 16 bytes: with K token-major four neighbouring lanes were in four cache lines, and the address unit takes them
// line by line.  us per step, token-major -> this order: 0.5B, 64 rows, contexts of 1050 781 -> 770; 1.5B, contexts of 710, 64
// rows 1775 -> 1729, 256 rows 2382 -> 2275; 64 x 768 scored tokens, 1.5B 142.5 -> 139.1 ms, 0.5B 48.6 -> 48.2.
__host__ __device__ __forceinline__ int k_page_at(int slot, int dim) {
  return ((((dim >> 5) * 2 + ((slot >> 2) & 1)) * 4 + ((dim >> 3) & 3)) * 8 + 4 * (slot >> 3) + (slot & 3)) * 8 + (dim & 7);
}
__host__ __device__ __forceinline__ int v_page_at(int slot, int dim) {
  return (((dim >> 4) * 2 + (slot >> 3)) * 16 + (dim & 15)) * 8 + (slot & 7);
}
// a lane's 16 bytes of a fragment within its page: lanes with l % 16 < 8 (K) or l < 32 (V) read the pair's first page
__device__ __forceinline__ int k_frag_at(int t, int kk, int lane) { return (((kk * 2 + t) * 4 + (lane >> 4)) * 8 + (lane & 7)) * 8; }
__device__ __forceinline__ int v_frag_at(int dt, int lane) { return ((dt * 2 + ((lane >> 4) & 1)) * 16 + (lane & 15)) * 8; }

// ---------------------------------------------------------------------------------------
// Device helpers
// ---------------------------------------------------------------------------------------
// A pair (a, b) rotated by (cos, sin), the rounding written out - one product rounded, then one fused multiply-add -
// so that every decode kernel that rotates gives the same bits whatever the code around the expression looks like
// (left to the compiler, which product is fused depends on the instruction order it happens to pick).
__device__ __forceinline__ float rot_first(float a, float b, float c, float s) { return __builtin_fmaf(a, c, -(b * s)); }
__device__ __forceinline__ float rot_second(float a, float b, float c, float s) { return __builtin_fmaf(b, c, a * s); }
// Sum of four squares, for the same reason.
__device__ __forceinline__ float sum_squares4(const float4& s) {
  return __builtin_fmaf(s.w, s.w, __builtin_fmaf(s.z, s.z, __builtin_fmaf(s.x, s.x, s.y * s.y)));
}
template <typename T> __device__ __forceinline__ float to_f32(T x) { return static_cast<float>(x); }
template <typename T> __device__ __forceinline__ T from_f32(float x) { return static_cast<T>(x); }
template <> __device__ __forceinline__ f16 from_f32<f16>(float x) { return (f16)fminf(fmaxf(x, -65504.f), 65504.f); }

// The wave's index inside its workgroup as a scalar (the same for every lane, and known to the compiler as such).
// Kernels guard matrix-core instructions with conditions on it ("has this wave another k step"); with the index in
// a vector register such a guard is a lane mask, the compiler may drop the branch around a short masked block, and a
// matrix-core instruction - which ignores the lane mask - then runs on registers that hold nothing.  A scalar index
// makes the guard a real branch.
__device__ __forceinline__ int wave_index(int thread_index) { return __builtin_amdgcn_readfirstlane(thread_index >> 6); }

// One value at an address that is the same for all lanes and that nothing writes while the kernel runs, through the scalar cache.
// (The compiler takes the vector path, and its wait for everything asked for before, once the kernel has stores in sight.)
__device__ __forceinline__ int load_uniform(const int* p) {
  return *(const __attribute__((address_space(4))) int*)(unsigned long long)p;
}

// The values of lanes l and l ^ 16 (l ^ 32) combined in every lane, through gfx950's lane-swap instructions
// (v_permlane16_swap / v_permlane32_swap: one vector-ALU instruction, no trip through LDS as the generic shuffle
// takes).  Both lanes of a pair combine (lower lane's value, upper lane's value) in that order.
typedef unsigned int lane_u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float max_xor16(float x) {
  const lane_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor32(float x) {
  const lane_u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor16(float x) {
  const lane_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_xor32(float x) {
  const lane_u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Lane q's value of every group of 4 lanes, in all four of them.
template <int Q> __device__ __forceinline__ float dpp_quad(float x) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), Q * 0x55, 0xf, 0xf, true));
}

__device__ __forceinline__ float wave_reduce_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_reduce_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Both halves of a 32 x 32 bit product in one instruction; written as two products the compiler keeps two.
__device__ __forceinline__ void mul_wide(uint32_t a, uint32_t b, uint32_t& hi, uint32_t& lo) {
  uint64_t p;
  asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(p) : "v"(a), "s"(b) : "vcc");
  hi = (uint32_t)(p >> 32);
  lo = (uint32_t)p;
}

// Philox4x32-10 (Salmon et al., SC'11): ten rounds on a 4-word counter with a 2-word key.
struct Philox4 { uint32_t x, y, z, w; };
__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    uint32_t hi0, lo0, hi1, lo1;
    mul_wide(c0, 0xD2511F53u, hi0, lo0);
    mul_wide(c2, 0xCD9E8D57u, hi1, lo1);
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  return Philox4{c0, c1, c2, c3};
}

// Standard Gumbel noise from one 32-bit random word: u = (2 (x >> 9) + 1) 2^-24 is strictly
// inside (0, 1) and exact in fp32; g = -ln(-ln u).
// Four values took 712 cycles of a wave, 411 of them in the logarithms, which is what bounded the LM head of 65 and more
// rows (118 us per step at 192 rows of the 0.5B decoder).  The arguments here are normal numbers (u >= 2^-24,
// 2^-24 < -ln u < 17), so the logarithm needs no range handling: 480 cycles.
// ln x = y ln 2 with y = log2 x of the hardware.  ln 2 = 0x1.62e42fefa39efp-1 is taken as c + c_low: its leading 23 bits and,
// rounded, the rest.  r = y c is rounded; fma(y, c, -r) is exactly what that rounding dropped (the two-product of an fma),
// and y c_low joins it before the one addition to r.  logf of AMD's open device library splits ln 2 the same way, and the
// result equals it in every bit for all 2^23 values of u.
__device__ __forceinline__ float ln_normal(float x) {
  constexpr float c = 0x1.62e42ep-1f, c_low = 0x1.efa39ep-25f;   // ln 2 = 0x1.62e42fefa39efp-1
  const float y = __builtin_amdgcn_logf(x), r = y * c;
  return r + __builtin_fmaf(y, c_low, __builtin_fmaf(y, c, -r));
}
__device__ __forceinline__ float gumbel_from_bits(uint32_t x) {
  const float u = (float)(2u * (x >> 9) + 1u) * 5.9604644775390625e-08f;
  return -ln_normal(-ln_normal(u));
}

// Noise for vocab entries 4*blk .. 4*blk+3 of (seed, seq, step): counter (blk, step, seq, 0),
// key = (seed low, seed high); entry v uses output word v % 4.
__device__ __forceinline__ void gumbel4(uint32_t seed_lo, uint32_t seed_hi, uint32_t seq, uint32_t step,
                                        uint32_t blk, float g[4]) {
  const Philox4 r = philox4x32_10(blk, step, seq, 0u, seed_lo, seed_hi);
  g[0] = gumbel_from_bits(r.x); g[1] = gumbel_from_bits(r.y);
  g[2] = gumbel_from_bits(r.z); g[3] = gumbel_from_bits(r.w);
}

// Running (max, sum of exp) pair of an online log-sum-exp.
struct LseAcc {
  float m, l;
  __device__ __forceinline__ void init() { m = -INFINITY; l = 0.f; }
  __device__ __forceinline__ void add(float z) {
    if (z > m) { l = l * __expf(m - z) + 1.f; m = z; } else { l += __expf(z - m); }
  }
  __device__ __forceinline__ void merge(float m2, float l2) {
    const float mn = fmaxf(m, m2);
    if (mn == -INFINITY) return;
    l = l * __expf(m - mn) + l2 * __expf(m2 - mn);
    m = mn;
  }
};

// Best perturbed score so far: larger y wins, equal y goes to the lower id.
struct BestAcc {
  float y, z; int id;
  __device__ __forceinline__ void init() { y = -INFINITY; z = 0.f; id = 0x7fffffff; }
  __device__ __forceinline__ void add(float y2, float z2, int id2) {
    if (y2 > y || (y2 == y && id2 < id)) { y = y2; z = z2; id = id2; }
  }
};

// ---------------------------------------------------------------------------------------
// Host-side launchers.  Every launcher enqueues on `st` and returns the launch's hipError_t.
// dtype: SAPO_DTYPE_F32 / SAPO_DTYPE_BF16 selects the element type T of weights/activations.
// ---------------------------------------------------------------------------------------
struct SampleParams {
  float temperature;
  uint32_t seed_lo, seed_hi;
  int max_new;            // row stride of out_tokens / out_logprobs
  const int* step;        // device: index of the token being sampled (0-based)
  const uint32_t* dyn;    // device, optional: {seed_lo, seed_hi, temperature bits} and, from word 15 on, the two output
                          // pointers, overriding the fields here (lets one captured graph serve calls that differ in these)
  int32_t* out_tokens;    // [S, max_new]
  float* out_logprobs;    // [S, max_new]
  // Stop token (optional): stop[0] = the token id that ends a sequence (< 0: none), stop[1] = number of
  // finished sequences, stop[2 + s] = length of sequence s once it has ended (0 while it runs).
  int* stop = nullptr;
  // Optional: arrival counter of the sampler's merge kernel.  When set, the last workgroup of the merge to
  // have read *step advances it (the step counter then needs no kernel of its own).
  int* arrivals = nullptr;
  // Optional, device: the sequence behind each row of the step (see RowMap::slot_seq).  The noise is keyed on
  // the sequence, and tokens, log-probs and lengths are written at the sequence's own rows.
  const int* slot_seq = nullptr;
  // Optional, device: a word that is non-zero once a decode step could not complete (see PersistCtl::fault).  From
  // then on the sampler emits token -1 with log-prob 0, so the failure is visible in the call's output.
  const unsigned* fault = nullptr;
  // Vocabulary size (0: unknown).  A sampled id outside [0, vocab) - what a row of NaN logits leaves behind, since no
  // score ever beats the initial one - is emitted as -1 and never used as an index.
  int vocab = 0;
};

// Optional per-kernel timing: when switched on, every launch carries two HIP events that take
// the kernel's start and end timestamps; the totals are read back per kernel symbol.  Off by
// default (the only cost is one branch per launch).
enum KernelId {
  KID_EMBED = 0, KID_RMSNORM, KID_GEMM_GENERIC, KID_ROPE_APPEND, KID_ATTN_GENERIC, KID_SWIGLU, KID_SAMPLE_ROWS,
  KID_SCORE_ROWS, KID_MISC, KID_GEMM_BIG, KID_LMHEAD_SCORE, KID_LMHEAD_SCORE_MERGE, KID_GEMM_SKINNY,
  KID_LMHEAD_SAMPLE, KID_LMHEAD_SAMPLE_MERGE, KID_DECODE_ATTN, KID_FLASH_ATTN, KID_GEMM_ROWS, KID_DECODE_LAYERS,
  KID_DECODE_ATTN_SHARED, KID_SMALL, KID_COUNT
};
extern bool g_prof_on;
// A pair of events for one profiled launch of kernel `kid` (recorded for sapo_profile_stop).
void prof_events(int kid, hipEvent_t* e0, hipEvent_t* e1);

// Every kernel launch of the library goes through here.  Normally a plain launch; while
// profiling, the launch carries two events that receive the kernel's own start and end
// timestamps (the figures a kernel trace reports, without the launch gaps around them).
template <typename... KArgs, typename... Args>
inline hipError_t launch(int kid, void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t smem, hipStream_t st,
                         Args... args) {
  static_assert(sizeof...(KArgs) == sizeof...(Args), "argument count mismatch");
  std::tuple<KArgs...> vals{static_cast<KArgs>(args)...};
  void* ptrs[sizeof...(KArgs) + 1];
  std::apply([&](auto&... v) { int i = 0; ((ptrs[i++] = (void*)&v), ...); }, vals);
  if (g_prof_on) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    prof_events(kid, &e0, &e1);
    return hipExtLaunchKernel((const void*)kernel, grid, block, ptrs, smem, st, e0, e1, 0);
  }
  return hipLaunchKernel((const void*)kernel, grid, block, ptrs, smem, st);
}

// The one place a sampled token is written.  A sequence that has emitted the stop token keeps
// emitting it with log-prob 0 (padding); the token returned is the one the next step embeds.
__device__ __forceinline__ int emit_token(const SampleParams& sp, int seq, int step, int token, float logprob) {
  if ((sp.fault && *sp.fault != 0u) || (sp.vocab > 0 && (unsigned)token >= (unsigned)sp.vocab)) {
    const size_t o = (size_t)seq * sp.max_new + step;
    sp.out_tokens[o] = -1;
    sp.out_logprobs[o] = 0.f;
    return 0;   // a valid id for the next step's embedding gather
  }
  if (sp.stop && sp.stop[0] >= 0) {
    int* len = sp.stop + 2 + seq;
    if (*len > 0) {
      token = sp.stop[0];
      logprob = 0.f;
    } else if (token == sp.stop[0]) {
      *len = step + 1;
      atomicAdd(sp.stop + 1, 1);
    }
  }
  const size_t o = (size_t)seq * sp.max_new + step;
  sp.out_tokens[o] = token;
  sp.out_logprobs[o] = logprob;
  return token;
}

__device__ __forceinline__ void resolve_sample_params(SampleParams& sp) {
  if (sp.dyn) {
    sp.seed_lo = sp.dyn[0];
    sp.seed_hi = sp.dyn[1];
    sp.temperature = __uint_as_float(sp.dyn[2]);
  }
}

__device__ __forceinline__ void resolve_outputs(SampleParams& sp) {
  if (sp.dyn) {
    sp.out_tokens = *(int32_t* const*)(sp.dyn + 15);
    sp.out_logprobs = *(float* const*)(sp.dyn + 17);
  }
}

// generic (shape-agnostic) kernels --------------------------------------------------------
hipError_t g_embed(int dtype, const int32_t* tokens, int tok_stride, const int* step, const void* embed,
                   float* h, int M, int d, hipStream_t st);
hipError_t g_rmsnorm(int dtype, const float* h, const float* gain, float eps, void* out, int M, int d,
                     const int* row_index, hipStream_t st);
enum GemmEpi { EPI_STORE_F32 = 0, EPI_ADD_F32 = 1 };
hipError_t g_gemm(int dtype, const void* A, const void* W, float* C, int M, int N, int K, int ldc, GemmEpi epi,
                  hipStream_t st);
hipError_t g_rope_append(int dtype, const float* qkv, const float2* rope, RowMap rm, KVCache kv, void* q_out,
                         int M, int n_q_heads, hipStream_t st);
hipError_t g_attention(int dtype, const void* q, RowMap rm, KVCache kv, void* out, int M, int n_q_heads,
                       int max_ctx, hipStream_t st);
hipError_t g_swiglu(int dtype, const float* gu, void* act, int M, int F, hipStream_t st);
hipError_t g_sample_rows(const float* logits, int n_prompt_rows, int G, int V, SampleParams sp, hipStream_t st);
hipError_t g_score_rows(const float* logits, int n_rows, int row_offset, int V, const int* row_seq_pos,
                        const int* n_rows_dev, const int32_t* tokens, int T, float* out_logprobs, hipStream_t st);
hipError_t g_advantages(const float* rewards, int S, int G, float* out, hipStream_t st);
// y = a x
hipError_t g_scale_f32(const float* x, float a, float* y, size_t n, hipStream_t st);
// x[m][n] += bias[n]
hipError_t g_add_row_bias(float* x, const float* bias, int M, int N, hipStream_t st);
// out[s] = len[s] if the sequence has stopped (len > 0), else max_new
hipError_t g_lengths_out(const int* len, int S, int max_new, int32_t* out, hipStream_t st);
// slot_seq[0 .. n_slots): the running sequences (len[s] == 0) in ascending order, then ended ones in ascending
// order as fill (n_slots <= S; the caller makes sure that at most n_slots sequences are running).
hipError_t g_compact_slots(const int* len, int S, int n_slots, int* slot_seq, hipStream_t st);
hipError_t g_assemble(const int32_t* local_tokens, const float* local_rewards, int n_local_pool, const int32_t* ext_tokens,
                      const float* ext_rewards, int n_ext_pool, int G, int T, int n_local, int n_ext, uint32_t seed_lo,
                      uint32_t seed_hi, int32_t* out_tokens, float* out_rewards, int* out_source, int* out_counts,
                      void* workspace, hipStream_t st);
size_t g_surrogate_workspace_bytes();
hipError_t g_surrogate_loss(const float* logp_new, const float* logp_old, const uint8_t* mask, const float* adv, int S, int T,
                            float eps_low, float eps_high, float* out_loss, float* out_dlogp, void* workspace,
                            hipStream_t st);
hipError_t g_page_table(int* pt, int n_seq, int pages_per_seq, int G, int full_prompt_pages, int n_prompts,
                        hipStream_t st);
hipError_t g_copy_partial_page(int dtype, KVCache kv, int n_prompts, int G, int page_idx, hipStream_t st);
// the same with one prompt length per prompt (device): page lens[p] / 16 of prompt p, if partly filled
hipError_t g_copy_partial_page_ragged(int dtype, KVCache kv, int n_prompts, int G, const int* lens, hipStream_t st);
// page table for prompts of different lengths: fp_max shared page slots per prompt, `own` pages per sequence
hipError_t g_page_table_ragged(int* pt, int n_seq, int pages_per_seq, int G, int fp_max, int own, int n_prompts,
                               const int* lens, hipStream_t st);
hipError_t g_fill_i32(int* p, int v, size_t n, hipStream_t st);
// counter += number of IEEE-half elements equal to +-65504 (the value the float -> half conversion clamps to) among the
// rows < rows_valid of buf; x32 != 0: buf is in 32-row fragment order (blocks of 32 rows x 16 k), else row-major
hipError_t g_count_half_at_limit(const void* buf, int rows_valid, int row_len, int x32, unsigned long long* counter,
                                 hipStream_t st);
hipError_t g_fill_f32(float* p, float v, size_t n, hipStream_t st);
struct RolloutBegin {
  int* step; int* stop; int* ctl;
  int n_ctl, S, stop_token;
  uint32_t seed_lo, seed_hi;
  float temperature;
  int32_t* out_tokens;
  float* out_logprobs;
};
hipError_t g_rollout_begin(const RolloutBegin& a, hipStream_t st);
hipError_t g_incr(int* p, hipStream_t st);
// Of sequences s0 .. s0 + ns - 1: how many rows each has among packed ones (packed_rows), and how many positions are scored
hipError_t g_packed_lens(const uint8_t* mask, int T, int s0, int ns, bool keep_aligned, int2* lens /*[ns]*/, hipStream_t st);
// RowMap::first [ns + 1] and ::packed [ns T] for those rows (kept aligned), and what g_masked_rows leaves (src_rows: packed
// rows); lens [ns]: scratch
hipError_t g_packed_rows(const uint8_t* mask, int T, int s0, int ns, const int* page_table, int pages_per_seq, int2* lens, int* first,
                         int2* packed, int* rows, int* src_rows, int* count, hipStream_t st);
// ... for prompts of lens[p] tokens, whose pages the first of G siblings' rows of the table name
hipError_t g_packed_prompts(const int* lens, int P, int G, const int* page_table, int pages_per_seq, int* first, int2* packed,
                            hipStream_t st);
hipError_t g_embed_packed(const int32_t* tokens, int T, int ns, const int* first, const void* embed, float* h, int d, hipStream_t st);
hipError_t g_masked_rows(const uint8_t* mask, int T, int s0, int ns, int* rows /*[ns*T,2]*/, int* src_rows /*[ns*T]*/,
                         int* count, hipStream_t st);
hipError_t g_rows_from_positions(const int* positions, int n, int T, int* src_rows, hipStream_t st);
// rows[p]: the row of prompt p's last position (lens, first: as in RowMap, or NULL)
hipError_t g_last_rows(int* rows, int P, int Lp, const int* lens, const int* first, hipStream_t st);
hipError_t g_gumbel(uint32_t seed_lo, uint32_t seed_hi, uint32_t seq, uint32_t step, uint32_t v0, int n, float* out,
                    hipStream_t st);

}  // namespace sapo

// =======================================================================================
// MFMA (bf16) kernels: weights live in "fragment order" so that a wave's operand load for one
// 32x32x16 MFMA step is one contiguous 1 KiB read:
//   Wp[((tile * (K/16) + ks) * 64 + lane) * 8 + e] = W[tile*32 + lane%32][ks*16 + (lane/32)*8 + e]
// =======================================================================================
namespace sapo {

int n_compute_units();   // of the device that was current at the first call

// Weights (fragment order: tiles of KS blocks of 1 KiB) of a later launch that extra workgroups of an earlier one bring into
// the L2s: the first ks1 blocks of every tile, the tiles of unit u (2^nt_log2 tiles) into the L2 of XCD u % 8.
struct Prefetch {
  const uint4* p = nullptr;
  int KS = 0, n_tiles = 0, nt_log2 = 0, ks1 = 0;   // ks1 = 0: nothing
};
// Measured on the two decoders of the workloads (0.5B, 1.5B), as the lines of the rules that choose between them
constexpr int kPrefetchKb = 28;       // blocks of 1 KiB per prefetching wave: at most (36 instead of 28 us per step + 5 to 32) ...
constexpr int kPrefetchKbFew = 6;     // ... beside gate/up of at most 16 rows ...
constexpr int kPrefetchKbRows = 18;   // ... and beside down of more than 64
// workgroups of `waves` waves for it, a multiple of 8
inline int prefetch_blocks(const Prefetch& pf, int waves, int per_wave) {
  const long kb = (long)pf.ks1 * pf.n_tiles;
  return (int)((kb + waves * per_wave - 1) / (waves * per_wave) + 7) / 8 * 8;
}
// Blocks per wave, from `lo` up, with which the workgroups of both fit into `room` compute units; none of them: otherwise.
// A launch's own workgroups and the prefetching ones belong on a compute unit each: one workgroup too many and two of them share
// one, the launch's own among them (us per step of a decode at the two sides of that line, attention launch: 0.5B, 64 rows, 248 and
// 264 workgroups 656, 691; 1.5B, 16 rows, 240 and 264 1098, 1173; 1.5B, 64 rows, 256 and 272 1619, 1678).
inline int prefetch_per_wave(const Prefetch& pf, const Prefetch& pf2, int waves, int room, int lo, int otherwise) {
  for (int per = lo; per <= kPrefetchKb; ++per)
    if (prefetch_blocks(pf, waves, per) + prefetch_blocks(pf2, waves, per) <= room) return per;
  return otherwise;
}
// All of a weight matrix, or the leading blocks of every tile where it is more than the L2s hold next to everything else
// (32 MB: 1.5B gate/up, 55 MB, of which half: 73.9 ms per call of 64 rows against 76.6 with all and 74.6 with none).
// The fraction is the same for every tile: leaving whole tiles out leaves the workgroups that read those as late as before.
inline Prefetch make_prefetch(const void* w, int KS, int n_tiles, int nt_log2) {
  Prefetch pf;
  pf.p = (const uint4*)w; pf.KS = KS; pf.n_tiles = n_tiles; pf.nt_log2 = nt_log2;
  const size_t cap_kb = 28 * 1024, kb = (size_t)KS * n_tiles;
  pf.ks1 = kb <= cap_kb ? KS : (int)(KS * cap_kb / kb);
  return pf;
}
// ---------------------------------------------------------------------------------------
// Prefetch workgroup: workgroups behind a launch's own that bring weights of a later launch into the L2s.
// A decode step is a chain of short launches, and the launches that stream (gate/up 17 MB, down 9 MB on the 0.5B
// decoder) wait for HBM from a standing start while the others (QKV, attention, O: 4 MB in 13 us) leave it idle.
// Lines that a kernel has read stay in its XCD's L2 across the kernel boundary, so the extra workgroups run on the XCD
// whose workgroups will read the weights (block ids are dealt round-robin): XCD x prefetches the tiles of the units
// x, x + 8, ... of the consumer.  0.5B, 64 rows: gate/up 8.8 -> 6.8 us, down 7.4 -> 6.3, attention (which carries
// gate/up's 17 MB on the compute units it leaves idle) 5.8 -> 7.0; on the wrong XCD the gain is lost.
// A wave asks for all of its blocks of 1 KiB at once and waits for them once: with 8 in flight and several rounds the
// launch that carries them got longer by what the consumer gained.  How many that are is the launch's to choose.  They go
// to LDS, all to the same KiB, which nobody reads: as register loads (18 or 28 of them unrolled) the role was most of a
// launch's code and up to half of its registers.  us per step, 0.5B, 24, 48 and 64 rows: 595, 613, 649 -> 591, 602, 640.
// ---------------------------------------------------------------------------------------
template <int NW>   // waves of a workgroup
__device__ __forceinline__ void prefetch_role(const Prefetch& pf, int block, int n_blocks, void* lds_1k) {   // lds_1k: 1 KiB of LDS
  const int xcd = block & 7, wv = (block >> 3) * NW + wave_index(threadIdx.x), nw = (n_blocks >> 3) * NW;   // waves per XCD
  const uint4* base = pf.p + (threadIdx.x & 63);
  const int n_units = pf.n_tiles >> pf.nt_log2, mine = ((n_units - xcd + 7) >> 3) << pf.nt_log2;   // tiles of this XCD
  const int span = pf.ks1, total = mine * span, nt1 = (1 << pf.nt_log2) - 1;
  for (int k = wv; k < total; k += nw) {
    const int m = k / span, tile = ((((m >> pf.nt_log2) << 3) + xcd) << pf.nt_log2) + (m & nt1);
    const uint4* p = base + ((size_t)tile * pf.KS + (k - m * span)) * 64;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                     (__attribute__((address_space(3))) void*)lds_1k, 16, 0, 0);
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the workgroup's LDS is given back when its waves have ended
}

// uint4 index of the chunk that holds x[tok][k .. k+7] (k a multiple of 8) in X16 order.
__host__ __device__ __forceinline__ size_t x16_chunk(int tok, int k, int KS) {
  return ((((size_t)(tok >> 6) * KS + (k >> 5)) * 4 + ((tok >> 4) & 3)) * 64) + (tok & 15) + 16 * ((k >> 3) & 3);
}

// the same in X32 order (32-token blocks, 16 k)
__host__ __device__ __forceinline__ size_t x32_chunk(int tok, int k, int KS) {
  return (((size_t)(tok >> 5) * KS + (k >> 4)) * 64) + (tok & 31) + 32 * ((k >> 3) & 1);
}

struct BigEpi {
  int mode;            // see enum below
  float* out_f32;      // STORE_F32 / ADD_F32: [M, ldc]
  int ldc;
  f16* out_act;        // SWIGLU: act, X32 order over F = N / 2
  // RMSNorm folded around the GEMM (a row's scale commutes with the contraction).  Consumer side: the
  // token operand holds x * gain without the row scale; the accumulators are multiplied by
  // rsqrt(sum of the row's ssq parts / norm_dim + eps) before the epilogue proper.
  const float* bias = nullptr;     // STORE_F32, optional: [N] added after the row scale
  const float* ssq_in = nullptr;   // [M, ssq_parts rounded up to a multiple of 4]; at most 16 parts
  int ssq_parts = 0;
  bool ssq_halves = false;         // every part as the two 64-feature halves it is the sum of: [M, 2 ssq_parts rounded up to a multiple of 4]
  float norm_dim = 0.f, eps = 0.f;
  // Producer side (ADD_F32 only): the updated residual row, times gain_next, goes out as half in X32
  // order (the next GEMM's operand), and its sum of squares in N / 128 parts per row.
  const float* gain_next = nullptr;   // [N]
  f16* xn_out = nullptr;
  float* ssq_out = nullptr;           // [M, N / 128 rounded up to a multiple of 4], or halves (m_gemm_writes_halves)
  const int* rows = nullptr;          // optional, device: how many rows there are, at most M
};
enum { BIG_STORE_F32 = 0, BIG_ADD_F32 = 1, BIG_SWIGLU = 2 };

// QKV projection with rotary embedding + KV append in the epilogue (head_dim 64 or 128)
struct QkvEpi {
  const float* ssq_in = nullptr;   // row scale of the folded norm, as in BigEpi
  int ssq_parts = 0;
  bool ssq_halves = false;
  float norm_dim = 0.f, eps = 0.f;
  const float* bias = nullptr;     // [N] optional
  const float2* rope = nullptr;    // [max_seq][hd / 2] (cos, sin)
  RowMap rm;
  KVCache kv;
  f16* q_out = nullptr;            // [M, Hq hd] rotated queries, half
  int n_q_heads = 0;
  const int* rows = nullptr;       // as in BigEpi
};
hipError_t m_gemm_qkv_rope(const void* Xp, const void* Wp, int M, int N, int K, const QkvEpi& epi, hipStream_t st);

constexpr int kPackRangeSlots = 512;   // pairs of range counters behind m_pack_weights' `range`
// One matrix [n_rows, K] (n_rows % 32 == 0, K % 64 == 0) into both fragment orders, or (dst32 NULL) n_rows floats into dst16.
struct PackTask {
  const void* src;
  uint4 *dst32, *dst16;
  int n_rows, K;
  int tile32, half;       // first 32-row tile; -1, or gate (0) / up (1) rows, 16 of each per tile
  int tile16, stride16;   // 16-row tile t goes to tile16 + t stride16
  int first_block;        // set by the launcher
};
hipError_t m_pack_weights(const PackTask* tasks, int n, unsigned* range, hipStream_t st);
// Xp: tokens in X32 fragment order (rows padded to a multiple of 32); Wp: weights in W32 order
// Whether a BIG_ADD_F32 launch of this size leaves its sums of squares in halves.
bool m_gemm_writes_halves(int M, int N);
hipError_t m_gemm_big(const void* Xp, const void* Wp, int M, int N, int K, BigEpi epi, hipStream_t st);
hipError_t m_rmsnorm_x32(const float* h, const float* gain, float eps, void* out, int M, int d, const int* row_index,
                         hipStream_t st, const int* rows = nullptr /* as in BigEpi */);
hipError_t m_lmhead_score(const void* Xp, const void* Wp, int max_rows, const int* n_rows_dev, int V, int K,
                          const int* row_seq_pos, const int32_t* tokens, int T, float* partials, float* out_logprobs,
                          hipStream_t st);
// rows src_rows[0 .. M - 1] (n_rows: *n_rows of them, at most M) of a residual [., d] and of an operand in X32 order over q, side by side
hipError_t m_gather_rows_x32(const int* src_rows, const int* n_rows, int M, const float* h, int d, const void* x, int q, float* h_out,
                             void* x_out, hipStream_t st);
size_t m_lmhead_score_partial_floats(int max_rows, int V);
// Fused LM head + sampler for any number of sequences and any K: Xp = final-normed rows in X32 order.
// partials: [m_lmhead_sample_big_groups(V)][n_rows][5].
int m_lmhead_sample_big_groups(int V);
hipError_t m_lmhead_sample_big(const void* Xp, const void* Wp, int n_rows, int V, int K, SampleParams sp, float* partials,
                               hipStream_t st);
// causal GQA attention over rows laid out [n_seq, rm.T] (block mode), K/V from the paged cache;
// q row-major, out in X32 order
hipError_t m_flash_attention(const void* q, RowMap rm, KVCache kv, void* out, int n_seq, int n_q_heads, hipStream_t st);

// FFN of a decode step of 65 .. 256 rows (kernels_rows.hip) ------------------------------------
// Xp: rows x gain in X32 order, ssq: their sums of squares [parts][s_pad] (an infinite part: a value was clamped), h, gain:
// what Xp was made of, read for the rows that half does not hold as they lie; Wp: W32 order, 16 gate and 16 up rows per block;
// act: X32 order over F
hipError_t r_gate_up(const void* Xp, const void* Wp, const float* ssq, int parts, int s_pad, int M, int F, int K, float eps, const float* h,
                     const float* gain, void* act, hipStream_t st);
// h += X W^T; xp = half(h * gain) in X16 order, ssq: [r_down_parts(d)][s_pad].  Xp in X32 order; pf: weights of a later launch
// that the product's launch brings into the L2s
constexpr int kRowSplits = 8;
int r_down_parts(int d);
size_t r_down_partial_floats(int M, int d);
hipError_t r_down(const void* Xp, const void* Wp, int M, int d, int K, float* partial, float* h, const float* gain, int s_pad, void* xp,
                  float* ssq, const Prefetch& pf, hipStream_t st);

// decode kernels (kernels_decode.hip) -------------------------------------------------------
constexpr int kMaxSsqParts = 96;   // parts of a row's sum of squares that d_gemm_skinny and d_lmhead_sample add up
enum { SKM_STORE = 0, SKM_RESID = 1, SKM_SWIGLU = 2, SKM_RESID_X32 = 3 };
struct SkinnyArgs {
  const uint4* Wp;        // weights, W16 fragment order [N/16][K/32][64]
  const uint4* Xp;        // tokens, X16 order [blocks][K/32][4][64]
  int N, K, n_rows;
  int s_pad;              // 64 * number of token blocks: row stride of the ssq arrays
  // STORE, SWIGLU: accumulators are scaled by rsqrt(sum_p ssq_in[p][tok] / norm_dim + eps)
  const float* ssq_in;    // [ssq_parts][s_pad]
  int ssq_parts;
  int norm_dim;
  float eps;
  float* out_f32;         // STORE: [n_rows, ldc]
  int ldc;
  const float* bias;      // STORE, optional: [N] added after the scale
  float* h;               // RESID: residual stream [n_rows, N], updated in place
  const float* gain_next; // RESID: gain of the norm that reads the updated residual [N]
  uint4* xp_out;          // RESID: half(h * gain_next), X16 order over K' = N; SWIGLU: act, X16 order over K' = N / 2
  Prefetch pf, pf2;       // weights of later launches to bring into the L2s
  int pf_blocks;          // workgroups of pf (set by the launcher)
  float* ssq_out;         // RESID: [N/16][s_pad] sums of h^2 over each 16-feature tile
};
hipError_t d_gemm_skinny(const SkinnyArgs& a, int mode, hipStream_t st);
// workgroup columns of a launch: parts of the sums of squares that RESID_X32 leaves
int d_skinny_units(int n_rows, int mode, int N, int K);
Prefetch d_prefetch_skinny(const void* w16, int n_rows, int mode, int N, int K);
hipError_t d_pack_rows_x16(const float* h, const float* gain, int M, int d, void* xp, float* ssq, hipStream_t st);
// Row m <- the embedding of the token that sequence m (slot_seq[m] when slot_seq is given) emitted at step *step - 1
hipError_t d_embed_x16(const int32_t* tokens, int tok_stride, const int* step, const void* embed, int M, int d,
                       const float* gain, float* h, void* xp, float* ssq, const int* slot_seq, hipStream_t st);
// d_gemm_skinny leaves the sums of squares of at most this many rows per group of 4 features ([tile][4][16 rows] in place
// of [tile][64 rows]) and expects them so
constexpr int kFewRows = 16;
bool d_lmhead_sample_supported(int K, int n_rows);
size_t d_lmhead_sample_partial_floats();
// Fused LM head + sampler for at most 64 sequences, followed by the merge that writes token and
// log-prob of the step and gathers the token's embedding row for the next step (h, X16 row with
// gain_first, one ssq part).
hipError_t d_lmhead_sample(const void* Wp, const void* Xp, int K, int V, const float* ssq, int ssq_parts, bool ssq_quarters, int s_pad,
                           float eps, int n_rows, SampleParams sp, float* partials, const void* embed,
                           const float* gain_first, float* h, void* xp_first, float* ssq_first, hipStream_t st);
// Merge of sampler partials [n_parts][row_stride][5] of n_rows sequences: token + log-prob of the step,
// then the embedding gather for the next step.
hipError_t d_lmhead_merge_embed(const float* partials, int n_parts, int row_stride, int n_rows, SampleParams sp,
                                const void* embed, int d, const float* gain_first, float* h, void* xp_first,
                                float* ssq_first, hipStream_t st);
// Decode attention with the prompt's pages read once per group of siblings (rows = P prompts x G siblings in order,
// every sequence at the same position, the siblings' page tables pointing at the same pages for the first
// 2 * prefix_pairs pages).  The launch then holds two kinds of workgroups: block ids 0 .. n_prefix - 1, one per
// (prompt, KV head), cover those pages for all siblings' query heads at once and leave per (row, query head) the
// unnormalised partial result (running max, sum, weighted values) in `pre`; the others, one per (row, KV head), cover
// the row's remaining tokens and fold the partial result in once the prefix workgroup's flag shows this launch's number.
struct ShareArgs {
  int G = 0;                  // siblings per prompt
  int prefix_pairs = 0;       // shared page pairs (32 tokens each); 0: no sharing
  int n_prefix = 0;           // P x KV heads
  float* pre = nullptr;       // [rows][n_q_heads][head_dim + 4]: m, l, -, -, o[head_dim]
  unsigned* flags = nullptr;  // [n_prefix], zero when the call begins; launch number = step * n_layers + layer + 1
  unsigned* fault = nullptr;  // set when a wait gave up
  int layer = 0, n_layers = 1;
  unsigned spin_ticks = 20000000u;   // bound of the wait in ticks of the 100 MHz wall clock
};
constexpr int kSharePrefixMaxColumns = 64;   // G x (query heads per KV head) the prefix workgroups can take
hipError_t d_decode_attention(const float* qkv, const float2* rope, RowMap rm, KVCache kv, void* out_x16, int S,
                              int n_q_heads, const ShareArgs* share, const Prefetch& pf, hipStream_t st);

// One decode step's layers as one persistent kernel (decode_persist.hip), up to 64 rows ----------------------
// Exchange counters between the resident workgroups; zeroed once at the start of a rollout call, then only growing
// (launch n since then starts from n x the arrivals of one launch).
struct PersistCtl {
  unsigned global;         // arrival groups that have completed a phase, summed over phases and launches
  unsigned pad0[63];
  unsigned group[8][64];   // one counter per arrival group, each in a 256-byte line of its own
  unsigned fault;          // set when a wait ran into its time limit: the step's results are not valid
  unsigned pad1[63];
  unsigned launches;       // launches of the persistent kernel since the counters were zeroed (moved on by the last
  unsigned pad2[63];       // workgroup to report the last phase of a launch)
};
struct PersistLayer {      // device table, one entry per layer (weights in W16 fragment order)
  const uint4 *wqkv, *wo, *wgu, *wdown;
  const float *bqkv, *ffn_norm, *gain_after;   // gain_after: the next layer's attention norm, or the final norm
};
struct PersistArgs {
  int n_layers, S, s_pad, d, q_dim, kv_dim, F, n_q_heads;
  float eps;
  const PersistLayer* layers;
  float* h;                // [S, d] residual stream
  float* qkv;              // [S, q + 2 kv]
  uint4* attn;             // X16 [s_pad, q]
  uint4* xa;               // X16 [s_pad, d]: QKV projection's operand (in: from the sampler's merge; out: for the LM head)
  uint4* xb;               // X16 [s_pad, d]: gate / up projection's operand
  uint4* act;              // X16 [s_pad, F]
  float* ssq_a;            // [d / 16][s_pad]; one part on entry
  float* ssq_b;            // [d / 16][s_pad]
  const float2* rope;
  RowMap rm;               // decode mode
  KVCache kv0;             // layer 0's cache
  size_t kv_layer_stride;  // bytes from a layer's K (V) pool to the next layer's
  PersistCtl* ctl;
  int v_qkv, v_o, v_gu, v_down;   // blocking of each GEMM phase (set by the launcher)
  unsigned spin_ticks;            // limit of one wait in ticks of the 100 MHz wall clock (set by the launcher)
};
size_t d_decode_layers_ctl_bytes();
bool d_decode_layers_supported(int S, int d, int q_dim, int kv_dim, int F, int head_dim, int n_kv_heads);
// kernel attributes and the residency check, once per process and outside any stream capture; the launch needs it
hipError_t d_decode_layers_prepare();
hipError_t d_decode_layers(PersistArgs args, int head_dim, hipStream_t st);

hipError_t g_gather_last_rows(const float* h, float* out, int S, int G, int Lp, int d, hipStream_t st);
// with per-prompt lengths (device): row p * Lp + lens[p] - 1
// first: RowMap::first where the rows are packed, or NULL
hipError_t g_gather_last_rows_ragged(const float* h, float* out, int S, int G, int Lp, const int* lens, const int* first, int d,
                                     hipStream_t st);

}  // namespace sapo
