"""The index arithmetic shared by set-up and kernels, on the CPU at mesh sizes no test system reaches."""
import os
import subprocess

import pytest

from paper_2010_09701_amd import build

HEADER = os.path.join(build.CSRC, "oefe_internal.h")

PROGRAM = r"""
#include "%s"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
  const int S = std::atoi(argv[1]), b[3] = {std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4])};
  std::printf("%%lld\n", (long long)oefe::slot_index(b[0], b[1], b[2], S));
}
"""


@pytest.fixture(scope="module")
def slot_index(tmp_path_factory):
    d = tmp_path_factory.mktemp("index")
    src = d / "index.cpp"
    src.write_text(PROGRAM % HEADER)
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    subprocess.run([hipcc, *build._flags(), str(src), "-o", str(d / "index")],
                   check=True, capture_output=True)
    return lambda *a: int(subprocess.run([str(d / "index"), *map(str, a)], check=True, capture_output=True,
                                         text=True).stdout)


@pytest.mark.parametrize("S", [12, 1290, 1291, 1935])  # 1290^3 < 2^31 < 1291^3; 1935: 3 slots of 645 cells
def test_slot_index(slot_index, S):
    for b in ((0, 0, 0), (S - 1, 0, 0), (1, S - 1, 0), (0, 2, S - 1), (S - 1, S - 1, S - 1)):
        assert slot_index(S, *b) == b[0] + S * (b[1] + S * b[2])
