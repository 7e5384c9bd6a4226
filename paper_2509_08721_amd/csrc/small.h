// Internal declarations of the small-decoder kernels (kernels_small.hip).
#pragma once
#include "common.h"

namespace sapo {

struct SmallLayer {   // device table, one entry per layer; matrices row-major as in the shape-generic path
  const void *wqkv, *wo, *wgu, *wdown;
  const float *attn_norm, *ffn_norm, *bqkv;
};
struct SmallModel {
  int L, d, hq, hkv, hd, F, V;
  float eps;
  const void* embed;
  const void* lm_head;
  const float* final_norm;
  const float2* rope;
  const SmallLayer* layers;
  void* pool;          // K and V of layer 0, K and V of layer 1, ...: pool_bytes each
  size_t pool_bytes;
};
struct SmallPrefill {
  const int32_t* tokens;   // [n_seq, T]
  int T;
  const int* lens;         // optional, device: positions of each sequence that count
  float* h_rows;           // [n_seq T, d] and
  void* q_rows;            // [n_seq T, Hq hd] (type T): a row's state between the launches of a long sequence
  int stage;               // set by the launcher
  float* h_last;           // rollout: [n_seq, d] residual row of the last position; NULL: scoring
  // scoring
  const uint8_t* mask;
  float* out_logprobs;     // [n_seq, T]
  float inv_t;
  const float* rewards;
  float* out_adv;          // [n_seq], groups of G
  int G;
};
struct SmallDecode {
  int P, Lp, G, N, ctx_max;
  const int* lens;
  const float* h_last;     // [P, d]
  float temperature;
  uint32_t seed_lo, seed_hi;
  int stop_token;          // < 0: none
  int32_t* out_tokens;     // [S, N]
  float* out_logprobs;
  int32_t* out_lengths;    // optional [S]
  bool lm_resident = false;   // set by the launcher: the LM head is kept in LDS
};
bool small_rows_fit(const SmallModel& m, size_t cache_rows, size_t prompt_rows, size_t io_elems);
bool small_prefill_fits(const SmallModel& m, int T);
bool small_decode_fits(const SmallModel& m, int ctx_max);
hipError_t small_prefill(int dtype, const SmallModel& m, const SmallPrefill& a, int n_seq, hipStream_t st);
hipError_t small_decode(int dtype, const SmallModel& m, const SmallDecode& a, int S, hipStream_t st);

// Group-relative advantages of one group, fp64; exactly 0 when all rewards are equal.
__device__ __forceinline__ void group_advantages(const float* __restrict__ rg, int G, float* __restrict__ out) {
  bool all_equal = true;
  double sum = 0.0;
  for (int i = 0; i < G; ++i) { sum += (double)rg[i]; all_equal = all_equal && (rg[i] == rg[0]); }
  if (all_equal) {
    for (int i = 0; i < G; ++i) out[i] = 0.f;
    return;
  }
  const double mu = sum / G;
  double var = 0.0;
  for (int i = 0; i < G; ++i) { const double dlt = (double)rg[i] - mu; var += dlt * dlt; }
  const double sd = sqrt(var / G);
  for (int i = 0; i < G; ++i) out[i] = (float)(((double)rg[i] - mu) / (sd + 1e-6));
}

}  // namespace sapo
