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
