"""Which form a small system's inner products take, and which single CG solves
run in one workgroup (csrc/slotrule.hpp), compiled on the host with g++:
against measured iteration times (us: copy, CSR lanes, multi-workgroup), a
choice may cost at most half as much again as the best one."""
import os
import shutil
import subprocess

import pytest

from helpers import ROOT

DRIVER = r"""
#include <cstdio>
#include "slotrule.hpp"
int main() {
    long long n, nnz, max_row;
    int lanes, threads, fp32;
    while (scanf("%lld %lld %lld %d %d %d", &n, &nnz, &max_row, &lanes, &threads, &fp32) == 6) {
        const bool one = ck::slot_one_lane(n, nnz, max_row, lanes, threads, fp32);
        printf("%d %d %d\n", one,
               ck::cg_in_one_workgroup(n, nnz, max_row, lanes, one, threads, fp32),
               ck::cg_in_one_workgroup(n, nnz, max_row, lanes, lanes == 1, threads, fp32));
    }
    return 0;
}
"""

# n, nnz, longest row, lanes, fp32 -> us per iteration from the copy, from the CSR
# arrays with the lanes, and on the multi-workgroup kernels
MEASURED = [
    (500, 1498, 3, 2, 0, 4.6, 6.8, 10.3),
    (4000, 11998, 3, 2, 0, 7.3, 9.2, 12.1),
    (8192, 24574, 3, 2, 1, 11.9, 12.9, 19.8),
    (2000, 9990, 15, 4, 0, 7.0, 10.8, 11.7),
    (6144, 55256, 21, 8, 0, 15.1, 32.4, 13.0),
    (1000, 16848, 28, 16, 0, 7.7, 13.3, 11.1),
    (4000, 67846, 33, 16, 0, 17.2, 38.7, 12.6),
    (4000, 67846, 33, 16, 1, 15.2, 33.3, 15.9),
    (4000, 202776, 75, 32, 0, 39.8, 76.2, 12.7),
    (6144, 615536, 139, 64, 1, 121.6, 260.5, 21.9),
    (1000, 4994, 1000, 4, 0, 100.9, 72.2, 33.9),
    (4000, 19994, 4000, 4, 1, 334.6, 243.5, 130.9),
    (1000, 18896, 1000, 16, 0, 100.1, 37.0, 21.6),
    (6144, 50414, 2006, 4, 0, 212.5, 584.8, 54.0),
    (4000, 15198, 204, 2, 0, 27.1, 70.6, 28.7),
    (6144, 19430, 502, 2, 1, 51.7, 68.1, 57.8),
    (4000, 78770, 1407, 16, 0, 148.0, 116.1, 21.1),
    (6144, 36478, 468, 4, 1, 45.5, 49.4, 24.7),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("slotrule")
    src, exe = d / "driver.cpp", d / "driver"
    src.write_text(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2411_10143_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)

    def ask(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows) + "\n"
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True)
        return [tuple(int(v) for v in line.split()) for line in out.stdout.splitlines()]
    return ask


def test_choices_against_measured_times(rule):
    got = rule([(n, nnz, mr, L, 1024, fp32) for n, nnz, mr, L, fp32, *_ in MEASURED])
    assert len(got) == len(MEASURED)
    for case, (one, inside, inside_lanes) in zip(MEASURED, got):
        copy, lanes, multi = case[5:]
        slot = copy if one else lanes
        assert (slot if inside else multi) <= 1.5 * min(copy, lanes, multi), case
        # a configuration that was given runs with its lanes, here or there
        assert (lanes if inside_lanes else multi) <= 1.5 * min(lanes, multi), case


def test_extremes(rule):
    got = rule([(8192, 8192 * 8192, 8192, 64, 1024, 0), (1, 1, 1, 1, 1024, 0),
                (1, 1, 1, 2, 256, 1), (5, 0, 0, 2, 1024, 0),
                (8000, 39994, 8000, 16, 1024, 0), (8000, 39994, 8000, 64, 1024, 1)])
    assert got[0][1:] == (0, 0)              # a dense matrix: never in one workgroup
    assert got[1] == (1, 1, 1)
    assert got[2][1:] == (1, 1) and got[3][1:] == (1, 1)
    assert got[4][0] == 0 and got[5][0] == 0   # one row of n: the lanes share it
