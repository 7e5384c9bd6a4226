// Index arithmetic that decides which addresses a kernel touches, in plain C++ without any HIP in it, so that a test on the
// host can walk it over the whole range of sizes.
#pragma once
#include <cstddef>
#include <cstdint>

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

// The small-decoder kernels index with 32 bits: K and V of a layer (cache_rows of kv values) and the call's tokens and
// outputs (io_elems of 4 bytes) stay below 2^31 bytes, the rows a long prompt keeps between launches (prompt_rows of d
// residual values, and of q query values) below 2^32 elements.
constexpr bool small_offsets_fit(uint64_t d, uint64_t q, uint64_t kv, uint64_t cache_rows, uint64_t prompt_rows, uint64_t io_elems) {
  return cache_rows * kv < (uint64_t)1 << 29 && io_elems < (uint64_t)1 << 29 &&
         prompt_rows * (d > q ? d : q) <= (uint64_t)1 << 32;
}

// Do two buffers of n bytes each share a byte?
constexpr bool overlap(uintptr_t a, uintptr_t b, size_t n) { return a < b ? b - a < n : a - b < n; }

}  // namespace sapo
