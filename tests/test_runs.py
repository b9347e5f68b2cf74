"""Rows taken in runs of a fixed length (csrc/fs_runs.h), up to the last row number there is: every row once, in order, and
no sum on the way that does not fit 32 bits."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_00194_amd", "csrc")

PROGRAM = """
#include <climits>
#include <cstdio>
#include <initializer_list>
#include "fs_runs.h"

template <int STEP>
static bool covers(int from, int to)
{
    long long next = from, runs = 0;
    fs::in_runs<STEP>(from, to, [&](int at, int left) {
        if (at != next || left != to - at || ++runs > 1 + ((long long)to - from) / STEP)
            __builtin_trap();
        next = at + (long long)(left < STEP ? left : STEP);
    });
    return next == (to > from ? to : from);
}

int main()
{
    for (int to : {0, 1, 5000, INT_MAX - 2048, INT_MAX - 2047, INT_MAX - 16, INT_MAX - 15, INT_MAX - 1, INT_MAX})
        for (int rows : {0, 1, 15, 16, 17, 2047, 2048, 2049, 4096, 6400})
            if (rows <= to && !(covers<STEP>(to - rows, to)))
                return printf("%d rows before %d\\n", rows, to), 1;
    return covers<STEP>(7, 3) ? 0 : 1;
}
"""


@pytest.mark.parametrize("step", [16, 2048])
def test_runs_end_at_the_last_row_number(tmp_path, step):
    src = tmp_path / "runs.cpp"
    src.write_text(PROGRAM.replace("STEP>(to", "%d>(to" % step).replace("covers<STEP>(7", "covers<%d>(7" % step))
    exe = str(tmp_path / "runs")
    subprocess.run(["g++", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CSRC, str(src), "-o", exe], check=True)
    done = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout + done.stderr
