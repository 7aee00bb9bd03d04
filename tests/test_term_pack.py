"""Packed terms of the weights (term_pack.h): every row's terms and exponent have bytes of their own, for any
number of rows (no GPU needed: the header is plain C++)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "term_pack.h"
int main(int argc, char** argv) {
  const int rows = std::atoi(argv[1]), K = std::atoi(argv[2]);
  std::vector<char> used(mg::pack2_bytes(rows, K));
  auto take = [&](size_t at, int n) {
    for (; n > 0; --n, ++at)
      if (at >= used.size() || used[at]++) { std::printf("byte %zu\\n", at); std::exit(1); }
  };
  for (int r = 0; r < rows; ++r) {
    for (int k8 = 0; k8 < K / 8; ++k8)
      for (int t = 0; t < 2; ++t)
        take(mg::pack_row(r, K, 2) + (size_t)k8 * 2 * mg::PACK_TERM + t * mg::PACK_TERM, 16);
    take(mg::pack_exponents_at(rows, K) + 4 * (size_t)r, 4);
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pack")
    (d / "pack.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2203_04738_amd", "csrc"),
                           "-o", str(d / "pack"), str(d / "pack.cpp")])
    return str(d / "pack")


@pytest.mark.parametrize("rows", [4, 8, 12, 20, 300, 304, 1004])
@pytest.mark.parametrize("K", [384, 408])
def test_terms_and_exponents_do_not_overlap(program, rows, K):
    r = subprocess.run([program, str(rows), str(K)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
