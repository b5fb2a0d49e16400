"""The index arithmetic with which the stem kernels copy image rows that are not
whole 16-byte units (csrc/rowunit.h), compiled for the host.

A band of ``rows`` image rows of ``rowlen`` values lies in memory ``skew`` values
after a 16-byte boundary and is read in units of ``vec`` values from that
boundary; a unit's first value is placed with unit_row, the rest follow by
counting.  Every value has to get the row and column that plain division gives.
"""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1907_01989_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "rowunit.h"
int main(int, char **argv) {
    const int vec = atoi(argv[1]);
    int bad = 0;
    for (int rowlen = 1; rowlen <= 70; ++rowlen)
        for (int skew = 0; skew < vec; ++skew)
            for (int rows = 1; rows <= 9; ++rows) {
                const int count = rows * rowlen, units = (skew + count + vec - 1) / vec;
                int placed = 0;
                for (int v = 0; v < units + 2; ++v) {     // (units past the band store nothing)
                    const int e0 = v * vec - skew;
                    int r = mgi::kern::unit_row(e0, rowlen, vec), c = e0 - r * rowlen;
                    for (int i = 0; i < vec; ++i) {
                        const int e = e0 + i;
                        if (e >= 0 && e < count) {
                            placed += 1;
                            bad += r != e / rowlen || c != e % rowlen;
                        }
                        if (++c == rowlen) { c = 0; ++r; }
                    }
                }
                bad += placed != count;
            }
    for (int rowlen : {4095, 4096, 32767})                // the longest rows a band can hold
        for (int e = -vec; e < 64 * rowlen; e += 61) {
            const int r = mgi::kern::unit_row(e, rowlen, vec), c = e - r * rowlen;
            bad += c < 0 || c >= rowlen;
        }
    printf("%d\n", bad);
    return 0;
}
"""


@pytest.mark.parametrize("vec", [4, 8])
def test_unaligned_rows_are_placed(tmp_path, vec):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1",
                           "-I", CSRC, str(src), "-o", str(exe)])
    assert int(subprocess.check_output([str(exe), str(vec)]).decode()) == 0
