"""Host-side rules of the direct eigensolver's dispatch, taken from the source."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1703_00387_amd import build as B


def _stages():
    """(rows a stage begins below, workgroups of its largest team, workgroups a CU holds), from the launches: a
    thread of EL complex elements, 512 threads, COLS columns; past 16 elements a CU holds one workgroup."""
    text = open(os.path.join(B.CSRC, "eig.hip")).read()
    out = []
    for cols, el in re.findall(r"tri_kernel<(\d+), (\d+)><<<", text):
        cols, el = int(cols), int(el)
        rows_per_wg = 8 * (el // (cols // 64))
        out.append((cols // 2, cols // rows_per_wg, 1 if el > 16 else 2))
    big = int(re.search(r"constexpr int kTriBigT = (\d+);", text).group(1))
    return out + [(2048, big, 1)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_every_team_of_a_matrix_taken_is_resident(tmp_path):
    text = open(os.path.join(B.CSRC, "common.h")).read()
    src = tmp_path / "r.cpp"
    src.write_text("#include <cstdio>\n#include <cstdlib>\nconstexpr int kEigMaxDim = 4096;\n" +
                   re.search(r"^inline int eig_max_rows\(.*?\}$", text, re.M | re.S).group(0) + "\n"
                   "int main(int c, char** v) { for (int i = 1; i < c; ++i) printf(\"%d\\n\", eig_max_rows(atoi(v[i]))); }\n")
    subprocess.run(["g++", "-o", str(tmp_path / "r"), str(src)], check=True)
    cus = [1, 16, 32, 38, 64, 128, 255, 256, 304]
    rows = subprocess.run([str(tmp_path / "r"), *map(str, cus)], capture_output=True, text=True, check=True).stdout.split()
    assert len(_stages()) == 7
    for n_cu, m in zip(cus, map(int, rows)):
        for lo, team, per_cu in _stages():
            assert m <= lo or team <= per_cu * n_cu, (n_cu, m, lo, team)
    assert int(rows[cus.index(256)]) == 4096       # the whole device takes every size
