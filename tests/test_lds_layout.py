"""LDS addresses of the kernels that have them in a host-only header, gone through lane by lane."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHORT = r'''
#include <cstdio>
#include "attn_short_layout.hpp"
template <int D> void columns() {
  for (int dt = 0; dt < (D + 1 + 15) / 16; ++dt)
    for (int piece = 0; piece < 4; ++piece) printf("%d %d %d %d\n", D, pab::SHORT_PITCH<D>, 16 * dt + 4 * piece, pab::short_v_column<D>(dt, piece));
}
int main() { columns<32>(); columns<72>(); }
'''


@pytest.fixture(scope="module")
def short_columns(tmp_path_factory):
    d = tmp_path_factory.mktemp("layout")
    (d / "short.cpp").write_text(SHORT)
    exe = str(d / "short")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2408_12588_amd", "csrc"), "-o", exe, str(d / "short.cpp")],
                   check=True, timeout=120)
    return [tuple(int(x) for x in line.split()) for line in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines()]


def test_value_operands_of_the_short_kernel_stay_in_their_rows(short_columns):
    """Every lane's four elements lie inside the row that it reads (hence inside the tile); the rows of V^T that matter, the D
    values and the row of the denominator, come from their own columns."""
    assert {D for D, *_ in short_columns} == {32, 72}
    for D, pitch, row, column in short_columns:
        assert 0 <= column and column + 4 <= pitch, (D, row, column)
        if row <= D:
            assert column == row, (D, row, column)
