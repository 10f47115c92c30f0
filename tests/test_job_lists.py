"""The surrogate-started build's lists of fold directions: a grid's jobs fill
them evenly, and so do the jobs of any one of its columns, whatever the grid's
width (list_of_job, compiled on the host)."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_26108_amd")
CODE = """
#include <stdio.h>
#include <stdlib.h>
#include "job_lists.h"
int main(int argc, char** argv) {
  const long n = atol(argv[1]);
  for (long j = 0; j < n; ++j) printf("%d\\n", chert::list_of_job(j, atoi(argv[2])));
}
"""


@pytest.fixture(scope="module")
def lists(tmp_path_factory):
    d = tmp_path_factory.mktemp("lists")
    src, exe = str(d / "m.cpp"), str(d / "m")
    with open(src, "w") as f:
        f.write(CODE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(PKG, "opcount"), "-I",
                    os.path.join(PKG, "csrc"), src, "-o", exe], check=True)
    return lambda jobs, n: np.array(subprocess.run([exe, str(jobs), str(n)], check=True,
                                                   capture_output=True, text=True).stdout.split(),
                                    dtype=int)


@pytest.mark.parametrize("nx,nz", [(64, 256), (128, 512), (256, 256), (101, 300), (320, 205),
                                   (1024, 64), (96, 128)])
def test_columns_are_spread_over_the_lists(lists, nx, nz):
    jobs = nx * nz
    n = max(1, min(64, jobs // 1024))
    part = lists(jobs, n)
    count = np.bincount(part, minlength=n)
    assert count.min() >= jobs // n - 1 and count.max() <= jobs // n + 1
    # a column's nz jobs in n lists: a list's share is binomial, six deviations
    per = part.reshape(nz, nx)
    most = max(np.bincount(per[:, x], minlength=n).max() for x in range(nx))
    assert most <= nz / n + 6.0 * np.sqrt(nz / n) + 1
