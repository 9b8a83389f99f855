"""Row offsets of the kernels (csrc/rows.h), compiled for the host: no GPU
needed."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2410_21607_amd", "csrc")


def run_host(tmp_path, body):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "t.cpp"
    src.write_text('#include "rows.h"\n#include <cstdio>\n#include <initializer_list>\nusing namespace sem;\nint main() {\n' + body + "\n}\n")
    exe = tmp_path / "t"
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_offsets_of_hanging_rows_are_dropped(tmp_path):
    """At every level of a row, a hanging point's offset is past the range of
    a state below 2 GiB and a unique node's is the row's own entry."""
    run_host(tmp_path, """
    const int nzn = 512, ldz = 512;
    for (int hh : {0, 1, 2, 511, 512, 3400000, (1 << 27) - 1}) {
        const unsigned r = row_offset(-(hh + 1), ldz);
        if (row_hanging(r) != hh) { std::printf("hanging point %d\\n", hh); return 1; }
        for (int kz = 0; kz < nzn; ++kz)
            if (r + 8u * unsigned(kz) < NOWHERE) { std::printf("in range: point %d level %d\\n", hh, kz); return 1; }
    }
    for (int g : {0, 1, 100000})
        if (row_offset(g, ldz) != 8u * 512u * unsigned(g)) { std::printf("node %d\\n", g); return 1; }
    return 0;""")


def test_level_pairs_stay_inside_the_row(tmp_path):
    """The pairs of levels that 16-byte loads take cover every level and none
    of the padding."""
    run_host(tmp_path, """
    for (int nzn = 2; nzn <= 600; ++nzn) {
        int last = -1;
        for (int k = 0; k < nzn; k += 2) {
            const int p = level_pair(k, nzn);
            if (p < 0 || p + 1 >= nzn) { std::printf("pair %d of %d levels\\n", p, nzn); return 1; }
            if (p > last + 1) { std::printf("level %d of %d left out\\n", last + 1, nzn); return 1; }
            last = p + 1;
        }
        if (last != nzn - 1) { std::printf("top of %d levels left out\\n", nzn); return 1; }
    }
    return 0;""")
