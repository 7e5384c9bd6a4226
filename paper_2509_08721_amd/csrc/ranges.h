// Index arithmetic that decides which addresses a kernel touches, in plain C++ without any HIP in it, so that a test on the
// host can walk it over the whole range of sizes.
#pragma once
#include <cstddef>
#include <cstdint>

#ifdef __HIP__
#define SAPO_HD __host__ __device__
#else
#define SAPO_HD
#endif

namespace sapo {

// Contraction of k_gemm_x3_tn over token rows [k_begin, k_end) in nst stages of ks rows.  The last stage ends at k_end, so
// the first one may begin in front of k_begin: only its masked loads (row()) may be used for it.  Stage s > 0 is requested
// row by row without a check; requests past the last stage ask for the last one again (its values are not used).  With one
// stage nothing is requested: that stage may have fewer than ks rows, and the rows in front of it need not exist.
struct StageRows {
  int k_begin, k_end, ks, nst, k_first;
  constexpr StageRows(int begin, int end, int stage_rows)
      : k_begin(begin), k_end(end), ks(stage_rows), nst((end - begin + stage_rows - 1) / stage_rows),
        k_first(end - nst * stage_rows) {}
  constexpr bool more() const { return nst > 1; }                      // is any stage requested ahead?
  constexpr int request(int s) const { return k_first + (s < nst ? s : nst - 1) * ks; }   // first row of a request, s >= 1
  constexpr bool in(int row) const { return row >= k_begin; }          // first stage: does the row count?
  constexpr int row(int i) const { return k_first + i > k_begin ? k_first + i : k_begin; }   // first stage: row i, clamped
};

// Block id -> (feature tile bx, token tile by) of the token-parallel products.  Block ids are dealt round-robin to the 8 XCDs, each
// with its own L2.  XCD c takes the c-th eighth of the tiles in this order: panels of 8 token tiles, in a panel blocks of 8
// feature tiles, in a block feature tiles fastest.  The 64 workgroups an XCD runs at a time then share 8 token tiles and 8
// feature tiles, and every XCD has as many tiles as the others.  Whole token tiles dealt to the XCDs (what this replaces) leave
// them unequal: 11 token tiles are two for three XCDs and one for five.  Scoring calls, us before and now, 0.5B: 9 x 301
// tokens (11 token tiles) 4542 -> 4024, 24 x 200 (19) 6414 -> 5653, 17 x 700 (47) 11715 -> 10949, 64 x 768 (192) within 0.2 %; 1.5B: 9 x 301
// 12258 -> 10277, 24 x 200 17066 -> 14602.  With the token tiles fastest in a panel 64 x 768 takes 1.4 % longer.
constexpr int tile_blocks(int NX, int NY) { return (NX * NY + 7) / 8 * 8; }   // blocks of the launch
// a / b for 0 <= a < 2^20, 0 < b < 2^19, from an approximation r of 1 / b within 2^-22 of it: (a + 1/2) / b lies 1 / (2 b) or more from the
// next integers, and what is computed within 2^-21 (a + 1/2) / b of it.
constexpr int quotient_by(int a, float r) { return (int)(((float)a + 0.5f) * r); }
// The same for 0 <= a < 2^31 - 2^19: what the approximation leaves is between -2^20 and 2^20.
constexpr int large_quotient_by(int a, int b, float r) {
  const int q = (int)((float)a * r), rest = a - q * b, more = quotient_by(rest < 0 ? -1 - rest : rest, r);
  return rest < 0 ? q - 1 - more : q + more;
}
SAPO_HD inline float reciprocal(int b) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_rcpf((float)b);
#else
  return 1.0f / (float)b;
#endif
}
SAPO_HD inline int quotient(int a, int b) { return quotient_by(a, reciprocal(b)); }
// What a workgroup executes before its first request counts: us per scoring call of 24 tokens, 6 layers of d_model 1024, with three of
// the compiler's divisions 286, with these quotients and no branch around the panels 284, as it is 263; 2709 tokens within 0.7 %.
SAPO_HD inline bool tile_of_block(int id, int NX, int NY, int& bx, int& by) {
  const int n = NX * NY, per = (n + 7) >> 3, j = id >> 3, t = (id & 7) * per + j;
  if (j >= per || t >= n) return false;
  int panel = 0, w = t, rows = NY;
  if (NY > 8) {
    panel = large_quotient_by(t, 8 * NX, reciprocal(8 * NX));
    w -= panel * 8 * NX;
    rows = NY - panel * 8 < 8 ? NY - panel * 8 : 8;
  }
  const int block = quotient(w, 8 * rows), v = w - block * 8 * rows, cols = NX - block * 8 < 8 ? NX - block * 8 : 8, y = quotient(v, cols);
  bx = block * 8 + v - y * cols;
  by = panel * 8 + y;
  return true;
}

// Groups that the LM-head scorer cuts the n_ft 128-feature tiles of the vocabulary into, each walked by one workgroup per row
// tile: as few as fill whole rounds of the `slots` workgroups in flight, of at most 32 tiles each.  The number of row tiles is
// that of the rows that are scored, which the device counts; what a row's log-prob is added up from does not depend on it
// (k_lmhead_score).  us per call with groups of 16 tiles, halved while half of the
// call's positions gave fewer than 512 workgroups, and with these: 0.5B, 24 x 200 tokens 5653, 5378; 9 x 301 4024, 3921 (the scorer 496 us
// with the row tiles dealt to the XCDs, now 312); 64 x 768 46.2 ms both; 1.5B, 24 x 200 14602, 14192.
struct ScoreGroups {
  int groups, tiles;   // their number, and the tiles of one (the last one may have fewer)
  SAPO_HD ScoreGroups(int n_ft, int row_tiles, int slots) : groups(0), tiles(1) {
    if (row_tiles <= 0 || n_ft <= 0) return;
    const int least = (n_ft + 31) / 32;
    const int rounds = quotient(least * row_tiles + slots - 1, slots), fill = quotient(slots * rounds, row_tiles);   // fill >= least
    const int most = fill < n_ft ? fill : n_ft;
    tiles = quotient(n_ft + most - 1, most);
    groups = quotient(n_ft + tiles - 1, tiles);
  }
};
// Largest number of workgroups of a call that scores up to max_rows rows
inline long score_most_workgroups(int n_ft, int max_rows, int slots) {
  long most = 0;
  for (int t = 1; t <= (max_rows + 255) / 256; ++t) {
    const long n = (long)ScoreGroups(n_ft, t, slots).groups * t;
    if (n > most) most = n;
  }
  return most;
}

// The small-decoder kernels index with 32 bits: K and V of a layer (cache_rows of kv values) and the call's tokens and
// outputs (io_elems of 4 bytes) stay below 2^31 bytes, the rows a long prompt keeps between launches (prompt_rows of d
// residual values, and of q query values) below 2^32 elements.
constexpr bool small_offsets_fit(uint64_t d, uint64_t q, uint64_t kv, uint64_t cache_rows, uint64_t prompt_rows, uint64_t io_elems) {
  return cache_rows * kv < (uint64_t)1 << 29 && io_elems < (uint64_t)1 << 29 &&
         prompt_rows * (d > q ? d : q) <= (uint64_t)1 << 32;
}

// Tile height (TJ blocks of 128 rows) and split of a packed product of the update (k_gemm_x3, k_gemm_x3_tn) with rows x cols
// outputs and KB steps of 16 along the contraction, in stages of `stage` steps; three products per value pair (NP 3, 2) or one.  A product whose
// output tiles fill the workgroups in flight badly (weight gradients: 49 .. 532 tiles; outputs d wide: 672 tiles on 512
// slots are 1.3 rounds run as 2) is split along the contraction where parts_cap (floats) allows it: each part writes its own
// product and k_sum_parts adds them in part order.  Taken are the height and number of parts with the least estimated time:
// rounds of resident workgroups (two per compute unit at 256 rows, three at 128) of so many steps, a tile's first requests
// and output, and the pass that adds the parts; among those whose chains are at most kChainSteps long.
// Why a limit: an accumulator loses a fraction of a unit in its last place at every step, so the error against 64 bits
// follows the longest chain, and the head's d-input product contracts over the vocabulary (9496 steps at 151936).  64 x 384
// tokens of the 0.5B decoder, three pieces: 4 parts of 2374 steps, the fastest by 2 % of the estimate, leave
// 1.5e-5 in the final norm's gradient and 2.4e-5 in the whole one, 16 parts of 594 steps 4.2e-6 and 1.5e-5; the update took
// 407.7 and 406.1 ms.
constexpr int kMaxSplits = 16, kChainSteps = 608;
struct X3Split { int TJ, parts, per_part; };
inline double x3_split_us(int NP, int TJ, int rows, int cols, int parts, int per_part) {
  const int gnx = (cols + 127) / 128, gty = ((rows + 127) / 128 + TJ - 1) / TJ;
  const long tiles = (long)gnx * gty, slots = TJ == 2 ? 512 : 768;
  // one 16-k step of a full round (measured: 1.35 PFLOP/s with three products, 0.9 with one; 10 % more for the small tile)
  const double step_us = (TJ == 2 ? 1.0 : 0.825) * 0.336 * (NP == 1 ? 1.0 : 3.0) * (NP == 1 ? 1.8 : 1.2);
  const long rounds = (tiles * parts + slots - 1) / slots;
  const double sum_us = parts > 1 ? 4.0 + (parts + 2) * 4e-6 * rows * cols : 0.0;   // at 1 MB per us
  return rounds * (per_part * step_us + (TJ == 2 ? 14.0 : 10.5)) + sum_us / 4.0;
}
inline X3Split x3_split(int NP, int rows, int cols, int KB, int stage, size_t parts_cap, int chain = kChainSteps) {
  X3Split best{2, 1, (KB + stage - 1) / stage * stage};
  double best_us = 0.0;
  for (int TJ = 2; TJ >= 1; --TJ)
    for (int s = 1; s <= kMaxSplits; ++s) {
      if (s > 1 && (KB / s < 16 || (size_t)s * rows * cols > parts_cap)) break;
      if ((KB + s - 1) / s > chain && s < kMaxSplits && (size_t)(s + 1) * rows * cols <= parts_cap) continue;
      const int per = ((KB + s - 1) / s + stage - 1) / stage * stage;
      if ((KB + per - 1) / per != s) continue;
      const double us = x3_split_us(NP, TJ, rows, cols, s, per);
      if (best_us == 0.0 || us < best_us * 0.98) {
        best_us = us;
        best = X3Split{TJ, s, per};
      }
    }
  return best;
}

// The same for an update that leaves rows out (leaves_rows_out): no chain is longer than with all of them (all_rows, all_KB; 32 steps and
// fewer are short anyhow), so that a gradient is no further off.  Chosen by the rows that are left, gate/up's d-input product had 608
// steps at 18209 of 24576 rows (0.5B, 64 x 384) in place of 204, and the gradient's error against 64 bits, three pieces, was 1.11e-5 where all
// rows left 7.2e-6 (7.2e-6 now; 48 x 300 5.4e-6, all rows 9.4e-6).
// With one and two pieces a product whose rows are the tokens is split exactly as with all of them, so that a row keeps its bits
// whatever is left out: a last bit decides how operands are rounded in all layers in front.  One piece, 21 x 301, the weights after
// one update against those of an update of all rows: 1.8e-3 off with splits of its own, 4e-6 with theirs, in the same time (35.3, 34.9 ms).
constexpr int kShortChain = 32;
inline X3Split x3_split_packed(int NP, int rows, int cols, int KB, int all_rows, int all_KB, int stage, size_t parts_cap) {
  X3Split all = x3_split(NP, all_rows, cols, all_KB, stage, parts_cap);
  if (rows == all_rows && KB == all_KB) return all;
  if (NP == 3 || KB != all_KB) {
    const int chain = all.per_part < kShortChain ? kShortChain : all.per_part < kChainSteps ? all.per_part : kChainSteps;
    return x3_split(NP, rows, cols, KB, stage, parts_cap, chain);
  }
  all.TJ = x3_split_us(NP, 1, rows, cols, all.parts, all.per_part) < 0.98 * x3_split_us(NP, 2, rows, cols, all.parts, all.per_part) ? 1 : 2;
  return all;
}

// Rows that a sequence of T positions has among packed rows when its last scored token is at `last` (0: it has none): the positions in
// front of it, which the token's log-prob depends on.
// The QKV launch writes 8 values of a page at once where a run of 8 slots lies within a tile of 64 rows, and two bytes at a time
// elsewhere.  An answer up to the row's end has T - 1 rows; for an even T they would leave every sequence behind it askew to the
// tiles, so a scoring pass (keep_aligned) takes the last position along: a call of such answers lies as it would without packing.  us per call not packed, with T - 1 and with T rows, 0.5B, every answer up to the row's end: 10 x 256 3396, 3484, 3418; 16 x 512
// 8505, 8640, 8538; 40 x 64 3326, 3406, 3345; 40 x 72 3745, 3773, 3722; 13 x 300 4774, 4810, 4790; 1.5B, 16 x 256 12790, 12950, 12894.  Answers that end anywhere are askew in
// any case; an even number of rows for each gains 0.3 % there, and loses 3 % where it begins another tile (9 x 301, 2048 rows -> 2052
// 3100 -> 3187).  Below 64 positions a row is more of a sequence than the alignment is worth: 8192 x 2 16738, 11913, 16698; 1000 x 8 8110, 7627,
// 8123; 600 x 16 9615, 8923, 9585; 400 x 32 11985, 11878, 11931.
SAPO_HD constexpr int packed_rows(int last, int T, bool keep_aligned) {
  return keep_aligned && T >= 64 && T % 2 == 0 && last == T - 1 ? T : last;
}

// Are there enough rows to leave out?  With a few fewer than a row tile of 128 a pass keeps its tiles, while aligned sizes become
// ragged ones, with blocks that are filled in part and fewer splits of the products over tokens.  So a sixteenth of the rows and
// at least `least` of them (needed 0: nothing depends on any row, all run as they lie).
// Prompts, a call of two tokens, all and packed, 0.5B: 72 of 1024 positions fewer 2345, 2352 us; 154 fewer 2335, 2299; 1.5B: 5500, 5515; 5477, 5262.
// Update, 0.5B, three pieces: 512 -> 440 rows 18.46, 18.63 ms; 640 -> 600 19.77, 20.05; 768 -> 720 20.51, 20.87; 512 -> 384 18.34, 17.43; 640 -> 505 4 % less; 1024
// -> 890 22.70, 22.53.  With one piece, a third of the work per row, it takes more rows: 1024 -> 890 16.78, 17.17; 768 -> 600 15.59,
// 16.05; 1152 -> 890 0.3 % more; 512 -> 300 3 % less; 2048 -> 1792 21.31, 20.30.
constexpr size_t kLeastPromptRows = 128;
constexpr size_t least_update_rows(int pieces) { return pieces == 1 ? 192 : 128; }
constexpr bool leaves_rows_out(size_t all, size_t needed, size_t least) {
  return needed > 0 && needed <= all && all - needed >= all / 16 && all - needed >= least;
}

// Blocks of k_embed_packed: sequences in x, four positions of a sequence each in y.  A grid's second dimension ends at 65535; a pass
// has up to 131072 sequences, and a sequence fewer than 4096 positions.
struct PackedEmbedGrid {
  unsigned x, y;
  constexpr PackedEmbedGrid(int n_seq, int T) : x((unsigned)n_seq), y((unsigned)(T + 3) / 4) {}
};

// Do two buffers of n bytes each share a byte?
constexpr bool overlap(uintptr_t a, uintptr_t b, size_t n) { return a < b ? b - a < n : a - b < n; }

}  // namespace sapo
