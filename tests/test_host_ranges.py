"""The index arithmetic of csrc/ranges.h, walked on the host over the sizes a kernel may meet."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not os.path.exists(CXX), reason="no C++ compiler")


def run(tmp_path, body):
    """Compiles `body` (which returns the number of mistakes and prints them) against the header and runs it."""
    src = tmp_path / "walk.cpp"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <vector>\n#include "ranges.h"\nusing namespace sapo;\n' + body)
    exe = str(tmp_path / "walk")
    subprocess.run([CXX, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2509_08721_amd", "csrc"),
                    str(src), "-o", exe], check=True)
    p = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert p.returncode == 0, p.stdout[-2000:]


def test_weight_gradient_products_read_only_their_own_token_rows(tmp_path):
    """k_gemm_x3_tn, every contraction length around its stages, split or not: each row of a part is multiplied once, and
    no row outside the part is read, also where one stage covers it all."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int ks : {16, 32})
    for (int K = 1; K <= 150; ++K)
      for (int split = ks; split <= 160; split += ks)
        for (int begin = 0; begin < K; begin += split) {
          const int end = K < begin + split ? K : begin + split;
          const StageRows r(begin, end, ks);
          std::vector<int> used(K, 0);
          auto read = [&](int row) {
            if (row < begin || row >= end) { if (++bad < 20) printf("ks %d K %d part [%d, %d): row %d read\n", ks, K, begin, end, row); return false; }
            return true;
          };
          for (int i = 0; i < ks; ++i)
            if (read(r.row(i)) && r.in(r.k_first + i)) ++used[r.row(i)];
          // the kernel: stage 1 before the loop, stage s + 2 within stage s, none in a last stage on its own
          if (r.more())
            for (int s = 1; s <= (r.nst % 2 ? r.nst : r.nst + 1); ++s)
              for (int i = 0; i < ks; ++i)
                if (read(r.request(s) + i) && s < r.nst) ++used[r.request(s) + i];
          for (int row = begin; row < end; ++row)
            if (used[row] != 1 && ++bad < 20) printf("ks %d K %d part [%d, %d): row %d used %d times\n", ks, K, begin, end, row, used[row]);
        }
  return bad != 0;
}
""")


def test_every_tile_has_one_block_and_the_xcds_share_alike(tmp_path):
    """Tiles of the token-parallel products over the blocks of a launch, and over a launch made for more token tiles than there
    are (the scorer's): each tile once, no XCD (id % 8) with more than an eighth, rounded up."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int NX : {1, 2, 7, 8, 9, 16, 36, 75, 76, 149, 1187})
    for (int NY = 0; NY <= 70; NY += NY < 20 ? 1 : 7)
      for (int more : {0, 5}) {
        std::vector<int> seen(NX * NY, 0);
        int per[8] = {};
        for (int id = 0; id < tile_blocks(NX, NY + more); ++id) {
          int bx = -1, by = -1;
          if (!tile_of_block(id, NX, NY, bx, by)) continue;
          if (bx < 0 || bx >= NX || by < 0 || by >= NY) { ++bad; printf("%d x %d block %d: %d %d\n", NX, NY, id, bx, by); continue; }
          ++seen[by * NX + bx];
          ++per[id & 7];
        }
        for (int s : seen) bad += s != 1;
        for (int p : per) bad += p > (NX * NY + 7) / 8;
      }
  return bad != 0;
}
""")


def test_quotients_by_an_approximate_reciprocal_are_exact(tmp_path):
    """Around multiples of b up to 2^20, and up to 2^31 - 2^19 for the large ones, with reciprocals as far off as quotient_by allows."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int b = 1; b <= 12000; b += b < 600 ? 1 : 61)
    for (double off : {-1.0, 0.0, 1.0}) {
      const float r = (float)((1.0 / b) * (1.0 + off * 1.8e-7));   // and a rounding: within 2^-22
      for (int q = 0; q * b < 1 << 20; q += 1 + q / 97)
        for (int a : {q * b - 1, q * b, q * b + b / 2})
          if (a >= 0 && a < 1 << 20 && quotient_by(a, r) != a / b) { if (!bad) printf("%d / %d\n", a, b); ++bad; }
      const long most = (1L << 31) - (1L << 19);
      for (long q = 0; q * b < most; q += 1 + q / 61)
        for (long a : {q * b - 1, q * b, q * b + b / 2, most - 1 - q})
          if (a >= 0 && a < most && large_quotient_by((int)a, b, r) != a / b) { if (!bad) printf("%ld / %d\n", a, b); ++bad; }
    }
  return bad != 0;
}
""")


def test_scorer_groups_cover_the_vocabulary_within_their_launch(tmp_path):
    """Every feature tile lies in one group, no group is empty or longer than 32 tiles, and the launch made for
    max_rows holds what any smaller number of rows asks for."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int n_ft : {1, 2, 8, 31, 32, 33, 64, 400, 1187, 2000})
    for (int slots : {512, 304})
      for (int max_rows : {1, 255, 256, 257, 2709, 49152}) {
        const long most = score_most_workgroups(n_ft, max_rows, slots);
        for (int rows = 0; rows <= max_rows; rows += rows < 600 ? 1 : 509) {
          const int t = (rows + 255) / 256;
          const ScoreGroups g(n_ft, t, slots);
          if (rows == 0) { bad += g.groups != 0; continue; }
          bad += g.tiles < 1 || g.tiles > 32 || g.groups * g.tiles < n_ft || (g.groups - 1) * g.tiles >= n_ft;
          bad += (long)g.groups * t > most;
          if (bad) { printf("%d tiles, %d slots, %d of %d rows: %d groups of %d\n", n_ft, slots, rows, max_rows, g.groups, g.tiles); return 1; }
        }
      }
  return 0;
}
""")


def test_buffers_that_share_a_byte_are_seen(tmp_path):
    """Which buffers the surrogate may not write while it reads them."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int a = 0; a < 12; ++a)
    for (int b = 0; b < 12; ++b)
      for (int n = 1; n < 8; ++n) {
        bool shared = false;
        for (int i = 0; i < n; ++i) for (int j = 0; j < n; ++j) shared |= a + i == b + j;
        if (overlap(a, b, n) != shared) { ++bad; printf("%d %d of %d bytes\n", a, b, n); }
      }
  return bad != 0;
}
""")


def test_small_decoder_offsets_stay_within_32_bits(tmp_path):
    """Whatever the rule lets through has its largest index below 2^32 (the kernels compute (row * heads + head) * head dim +
    dim and row * width + column in unsigned 32 bits), over the model widths and batch sizes a rollout call accepts."""
    run(tmp_path, r"""
int main() {
  int bad = 0, let = 0, held = 0;
  const uint64_t lim = (uint64_t)1 << 32;
  for (uint64_t d : {4, 64, 128, 252, 256, 260, 512, 4096})
    for (uint64_t q : {4, 64, 256, 300, 1024})
      for (uint64_t kv : {4, 8, 32, 64, 256})
        for (int lg = 0; lg <= 24; ++lg)                 // prompt positions: at most 2^24
          for (uint64_t less : {0, 1}) {
            const uint64_t rows = ((uint64_t)1 << lg) - (lg ? less : 0);
            for (uint64_t gen : {1u, 1u << 10, 1u << 20, 1u << 26}) {   // generated positions
              const uint64_t cache = rows + gen, io = rows > gen ? rows : gen;
              if (!small_offsets_fit(d, q, kv, cache, rows, io)) { ++held; continue; }
              ++let;
              if (rows * d > lim || rows * q > lim || cache * kv > lim || io > lim) { ++bad; printf("d %d q %d kv %d rows %d\n", (int)d, (int)q, (int)kv, (int)rows); }
            }
          }
  if (small_offsets_fit(260, 8, 8, 1 << 24, 1 << 24, 1 << 24)) { ++bad; printf("2^24 rows of 260 let through\n"); }
  if (!small_offsets_fit(64, 64, 16, 1 << 24, 1 << 24, 1 << 24)) { ++bad; printf("2^24 rows of 64 held back\n"); }
  printf("%d let through, %d held back\n", let, held);
  return bad != 0 || !let || !held;
}
""")


def test_products_of_the_update_are_split_without_long_chains(tmp_path):
    """x3_split over the products of small and large decoders: the parts cover the contraction, none is empty, and no
    accumulator's chain is longer than 608 steps (one stage's rounding apart) unless 16 parts or the buffer for the parts do
    not allow it."""
    run(tmp_path, r"""
int main() {
  int bad = 0, limited = 0;
  const size_t caps[] = {0, (size_t)1 << 20, (size_t)8 * 2 * 4864 * 896, (size_t)8 * 2 * 8960 * 1536};
  for (int NP = 1; NP <= 3; ++NP)
    for (int stage : {NP == 3 ? 1 : NP == 2 ? 2 : 4, NP == 1 ? 2 : 1})
      for (int rows : {1, 64, 130, 896, 1152, 2500, 4352, 9728, 24576, 151936})
        for (int cols : {48, 896, 1536, 4864, 17920})
          for (int K : {1, 16, 100, 896, 4864, 9728, 9744, 17920, 24576, 151936, 300000})
            for (size_t cap : caps) {
              const int steps = (K + 15) / 16, KB = (steps + stage - 1) / stage * stage;
              const X3Split s = x3_split(NP, rows, cols, KB, stage, cap);
              const size_t out = (size_t)rows * cols;
              const bool covers = s.per_part % stage == 0 && (long)s.per_part * s.parts >= KB && (long)s.per_part * (s.parts - 1) < KB;
              const bool fits = s.parts == 1 || s.parts * out <= cap;
              const bool could = s.parts < kMaxSplits && (s.parts + 1) * out <= cap;
              const bool chain = s.per_part < kChainSteps + stage || !could;
              limited += s.per_part >= kChainSteps + stage;
              if (!covers || !fits || !chain || s.TJ < 1 || s.TJ > 2) { if (++bad < 20) printf("NP %d stage %d %d x %d K %d cap %zu: TJ %d, %d parts of %d\n", NP, stage, rows, cols, K, cap, s.TJ, s.parts, s.per_part); }
            }
  const X3Split head = x3_split(3, 4352, 896, 9496, 1, caps[2]);
  if (head.per_part > kChainSteps) { ++bad; printf("head: %d parts of %d\n", head.parts, head.per_part); }
  return bad != 0;
}
""")


def test_packed_embedding_grid_takes_every_number_of_sequences(tmp_path):
    """k_embed_packed: a block for every four positions of every sequence, in a grid whose second dimension is at most 65535."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int T : {1, 2, 3, 4, 5, 127, 300, 3583, 3584})
    for (int n : {1, 2, 65535, 65536, 65537, 131072, 1 << 20}) {
      const PackedEmbedGrid g(n, T);
      if (g.x != (unsigned)n || g.y * 4 < (unsigned)T || g.y > 65535 || (g.y - 1) * 4 >= (unsigned)T) { ++bad; printf("%d x %d: %u %u\n", n, T, g.x, g.y); }
    }
  return bad != 0;
}
""")


def test_packed_rows_hold_the_scored_tokens_prefix_and_full_answers_stay_aligned(tmp_path):
    """packed_rows: the positions in front of the last scored token, none for a sequence without one.  In a scoring pass an answer up
    to the end of a row of an even number of positions, 64 and more, keeps the last one too; no other row does."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int T = 1; T <= 700; ++T)
    for (int last = 0; last < T; ++last) {
      const bool full = T >= 64 && T % 2 == 0 && last == T - 1;
      if (packed_rows(last, T, true) != (full ? T : last) || packed_rows(last, T, false) != last) { ++bad; printf("T %d last %d: %d\n", T, last, packed_rows(last, T, true)); }
    }
  return bad != 0;
}
""")


def test_rows_are_left_out_only_where_a_tile_of_them_goes(tmp_path):
    """leaves_rows_out: never where nothing is needed, never for fewer rows than a row tile or a sixteenth, and once enough for some
    number of needed rows, enough for every smaller one."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  for (int pieces : {1, 2, 3})
    for (size_t all = 1; all <= 4200; all += all < 300 ? 1 : 37) {
      const size_t least = least_update_rows(pieces);
      if (leaves_rows_out(all, 0, least) || leaves_rows_out(all, all, least) || leaves_rows_out(all, all + 1, least)) { ++bad; printf("%zu: ends\n", all); }
      bool before = true;
      for (size_t needed = 1; needed < all; ++needed) {
        const bool out = leaves_rows_out(all, needed, least);
        if (out && (all - needed < 128 || (all - needed) * 16 < all - 15)) { ++bad; printf("%zu needed of %zu\n", needed, all); }
        if (out && !before) { ++bad; printf("%zu of %zu: not below\n", needed, all); }
        before = out;
      }
    }
  return bad != 0;
}
""")


def test_products_of_packed_updates_add_up_as_with_all_rows(tmp_path):
    """x3_split_packed: a product of an update that leaves rows out covers its contraction, fits the parts' buffer and adds up no
    chain longer than the same product with all rows does (32 steps and fewer apart).  With one and two pieces one whose rows are the
    tokens has the parts that it has with all rows (a row keeps its bits); with all rows it is x3_split."""
    run(tmp_path, r"""
int main() {
  int bad = 0;
  const int shapes[][3] = {{896, 1152, 9728}, {1536, 2048, 17920}, {64, 128, 384}};   // d, q + 2 kv, 2 F
  for (const auto& sh : shapes) {
    const int d = sh[0], nqkv = sh[1], F2 = sh[2];
    const size_t most = (size_t)F2 * d, cap = 8 * (most > (size_t)192 * 128 * 128 ? most : (size_t)192 * 128 * 128);
    for (int NP : {1, 2, 3})
      for (int all = 256; all <= 40000; all += all < 2000 ? 97 : 1531)
        for (int left = all; left >= 1; left -= left > 2000 ? 911 : left > 64 ? 61 : 1) {
          auto check = [&](int rows, int all_rows, int cols, int KB, int all_KB, int stage, size_t parts_cap) {
            const X3Split a = x3_split(NP, all_rows, cols, all_KB, stage, parts_cap);
            const X3Split s = x3_split_packed(NP, rows, cols, KB, all_rows, all_KB, stage, parts_cap);
            const bool same = rows != all_rows || KB != all_KB || (s.TJ == a.TJ && s.parts == a.parts && s.per_part == a.per_part);
            const bool covers = s.parts * s.per_part >= KB && (s.parts - 1) * s.per_part < KB;
            const bool fits = s.parts == 1 || (size_t)s.parts * rows * cols <= parts_cap;
            const int most_steps = a.per_part > kShortChain ? a.per_part : kShortChain;
            const bool as_all = NP == 3 || KB != all_KB ? s.per_part <= most_steps : s.parts == a.parts && s.per_part == a.per_part;
            if (!same || !covers || !fits || !as_all) {
              if (++bad < 20) printf("NP %d rows %d of %d cols %d steps %d of %d: %d x %d, with all %d x %d\n", NP, rows, all_rows, cols, KB, all_KB, s.parts, s.per_part, a.parts, a.per_part);
            }
          };
          const int st = NP == 1 ? 4 : 2, st_tn = NP == 1 ? 2 : 1;
          auto steps = [](int K) { return (K + 63) / 64 * 4; };
          // d-input and forward products, split or not: the tokens are rows
          for (size_t c : {cap, (size_t)0}) {
            check(left, all, d, steps(F2), steps(F2), st, c);
            check(left, all, d, steps(F2 / 2), steps(F2 / 2), st, c);
            check(left, all, d, steps(nqkv), steps(nqkv), st, c);
            check(left, all, F2 / 2, steps(d), steps(d), st, c);
            check(left, all, F2, steps(d), steps(d), st, c);
          }
          // weight gradients: the tokens are contracted over
          check(F2, F2, d, steps(left), steps(all), st, cap);
          check(d, d, F2 / 2, steps(left), steps(all), st, cap);
          check(nqkv, nqkv, d, (left + 15) / 16, (all + 15) / 16, st_tn, cap);
        }
  }
  return bad != 0;
}
""")
