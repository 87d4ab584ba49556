"""The host's rules (csrc/rules.h), compiled for the CPU and evaluated here."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2510_25991_amd", "csrc")


def evaluate(tmp_path, body):
    """Output lines of a C++ main() with this body."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include "rules.h"\nusing namespace ddst;\n'
                   "int main() {\n" + body + "\n  return 0;\n}\n")
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()


def test_dot_workspace_holds_every_shorter_vector(tmp_path):
    """A workspace sized for one length serves every shorter one (a solve of
    several loads works on stacked vectors and on single ones)."""
    bad = evaluate(tmp_path, """
  size_t most = 0;
  for (size_t len = 1; len <= 400000; ++len) {
    most = std::max(most, dot_chunks(len));
    if (dots_part_len(len, 3) < 3 * most) { std::printf("%zu\\n", len); break; }
  }""")
    assert bad == []


@pytest.mark.parametrize("dim,n,slabs,sym,outer", [
    (2, 1151, 2, 0, 0), (2, 1151, 4, 0, 0), (2, 1535, 4, 0, 0), (2, 2047, 4, 1, 0),
    (3, 39, 4, 0, 0), (3, 47, 4, 1, 0), (2, 1023, 16, 0, 0), (2, 1023, 32, 1, 0),
    (2, 1023, 32, 0, 1), (2, 1023, 64, 1, 1), (2, 1535, 16, 0, 1), (2, 2047, 16, 0, 1),
    (3, 63, 8, 1, 1), (2, 767, 64, 0, 0)])
def test_outer_blocks_take_the_faster_way(tmp_path, dim, n, slabs, sym, outer):
    """Builds whose two ways were measured (the matrices of all sweeps at once)."""
    ld = (n ** (dim - 1) + 127) // 128 * 128
    got = evaluate(tmp_path, 'std::printf("%%d %%d", (int)outer_blocks(%d, %d, 4, %s), '
                   "(int)outer_blocks(%d, %d, 8, %s));"
                   % (2 * slabs - 1, ld, "true" if sym else "false",
                      2 * slabs - 1, ld, "true" if sym else "false"))
    assert got == [str(outer), "0"]


@pytest.mark.parametrize("njobs,ld,big", [
    (900, 128, 0), (225, 384, 0), (100, 640, 0), (94, 896, 0), (36, 1152, 0), (25, 1408, 0),
    (1, 1024, 0), (4, 256, 0), (33, 1024, 0), (60, 1024, 1), (188, 1024, 1), (225, 512, 1),
    (16, 1920, 1), (4000, 2048, 1)])
def test_products_take_the_faster_tiles(tmp_path, njobs, ld, big):
    got = evaluate(tmp_path, f'std::printf("%d", (int)gemm_big_tiles({njobs}, {ld}));')
    assert got == [str(big)]


@pytest.mark.parametrize("rows,most", [(1, 2), (32, 2), (64, 2), (65, 4), (128, 4)])
def test_rows_in_flight_of_the_sampled_product(tmp_path, rows, most):
    got = evaluate(tmp_path, f'std::printf("%d", hbs_rows_in_flight({rows}));')
    assert got == [str(most)]


@pytest.mark.parametrize("njobs,ld,wide", [(1, 128, 0), (64, 512, 0), (32, 1024, 0), (6, 2304, 0),
                                           (64, 1024, 1), (128, 1024, 1), (16, 2048, 1),
                                           (40000, 16256, 1)])
def test_columns_of_the_matrix_vector_product(tmp_path, njobs, ld, wide):
    got = evaluate(tmp_path, f'std::printf("%d", (int)gemv_wide({njobs}, {ld}));')
    assert got == [str(wide)]


def test_pivots_share_cus_beyond_one_each(tmp_path):
    got = evaluate(tmp_path, 'std::printf("%d %d %d", (int)pivots_share_cus(63), '
                             "(int)pivots_share_cus(256), (int)pivots_share_cus(257));")
    assert got == ["0", "0", "1"]


@pytest.mark.parametrize("njobs,ld,esz,rows", [(16, 1024, 4, 0), (64, 512, 8, 0), (32, 1024, 4, 0),
                                               (32, 1024, 8, 1), (64, 768, 8, 1),
                                               (16, 2048, 4, 1), (4, 3968, 4, 1)])
def test_order_of_the_transposed_product(tmp_path, njobs, ld, esz, rows):
    got = evaluate(tmp_path, f'std::printf("%d", (int)gemv_t_rows({njobs}, {ld}, {esz}));')
    assert got == [str(rows)]
