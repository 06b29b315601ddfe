"""Which tile a launch of the fused kernels takes: the host rule, compiled by itself."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2501_19392_amd", "csrc")
PROGRAM = """
#include <cstdio>
#include "tile_choice.h"
using namespace aquakv;
int main() {
  long long n, s;
  int d;
  char kind;                                       // encode with a grid, predictions, others; others without a tile of two heads: O
  while (std::scanf("%lld %lld %d %c", &n, &s, &d, &kind) == 4)
    std::printf("%d\\n", tile_rows(n, s, d, kind != 'O', kind == 'e' ? kSearchRound192 : kind == 'p' ? kNoRound192 : kRound192));
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("choice")
    (d / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(d / "t"), str(d / "t.cpp")], check=True)

    def ask(calls):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        return [int(x) for x in subprocess.run([str(d / "t")], input=text, check=True, capture_output=True, text=True).stdout.split()]
    return ask


UP_TO_8192 = [(1, 32), (1024, 32), (1025, 64), (2048, 64), (2049, 96), (3072, 96), (3073, 128), (4096, 128), (4097, 192), (6144, 192), (6145, 0), (8192, 0),
              (8193, 320), (10240, 320)]


@pytest.mark.parametrize("kind,beyond", [
    ("e", [(10241, 192), (12288, 192), (12289, 0), (16385, 192), (18433, 320), (20481, 0), (32769, 192), (36864, 192), (36865, 0), (49153, 0)]),
    ("o", [(10241, 0), (16384, 0), (16385, 192), (18432, 192), (18433, 320), (20480, 320), (20481, 0), (32769, 0), (49153, 0), (65536, 0)]),
    ("O", [(10241, 192), (12288, 192), (12289, 0), (16385, 192), (18433, 320), (24577, 0), (32769, 0)]),
    ("p", [(10241, 0), (16385, 320), (18433, 320)])])
def test_rows_of_8_heads(rows, kind, beyond):
    """(tokens, rows), 0: 256 rows; 8 heads, at the ends of ranges"""
    edges = UP_TO_8192 + beyond
    assert rows((1, t, 1024, kind) for t, _ in edges) == [r for _, r in edges]


def test_rows_of_sequences(rows):
    """The shapes that the tests of scores on 192 rows in several rounds run, and many short sequences"""
    assert rows([(16, 1100, 1024, "O"), (3, 3500, 1024, "O"), (5, 3300, 1024, "O"), (5, 3300, 1024, "o")]) == [192] * 4
    assert rows([(16, 33, 1024, "o"), (1000, 33, 1024, "o"), (1, 33000, 384, "e")]) == [32, 0, 0]
