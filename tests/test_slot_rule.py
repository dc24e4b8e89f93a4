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
    int lanes, threads, fp32, m;
    while (scanf("%lld %lld %lld %d %d %d %d", &n, &nnz, &max_row, &lanes, &threads, &fp32,
                 &m) == 7) {
        const bool one = ck::slot_one_lane(n, nnz, max_row, lanes, threads, fp32);
        auto inside = [&](bool o) {   // m = 0: CG
            return m == 0 ? ck::cg_in_one_workgroup(n, nnz, max_row, lanes, o, threads, fp32)
                          : ck::gmres_in_one_workgroup(n, nnz, max_row, m, lanes, o, threads, fp32);
        };
        printf("%d %d %d\n", one, inside(one), inside(lanes == 1));
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
    got = rule([(n, nnz, mr, L, 1024, fp32, 0) for n, nnz, mr, L, fp32, *_ in MEASURED])
    assert len(got) == len(MEASURED)
    for case, (one, inside, inside_lanes) in zip(MEASURED, got):
        copy, lanes, multi = case[5:]
        slot = copy if one else lanes
        assert (slot if inside else multi) <= 1.5 * min(copy, lanes, multi), case
        # a configuration that was given runs with its lanes, here or there
        assert (lanes if inside_lanes else multi) <= 1.5 * min(lanes, multi), case


# n, nnz, longest row, lanes, fp32, m -> us a GMRES step in one workgroup, on the
# multi-workgroup kernels, and before the vectors were on the chip
GMRES = [
    (4, 14, 4, 1, 0, 30, 28.0, 36.1, 26.8), (4, 14, 4, 1, 1, 10, 11.1, 30.4, 15.6),
    (30, 88, 3, 2, 1, 1, 11.4, 26.1, 20.1), (30, 144, 30, 4, 1, 5, 11.6, 17.0, 16.1),
    (100, 298, 3, 2, 0, 1, 14.4, 26.1, 24.3), (100, 298, 3, 2, 0, 10, 17.0, 15.9, 20.2),
    (100, 298, 3, 2, 1, 10, 11.1, 14.4, 16.1), (100, 298, 3, 2, 1, 30, 18.7, 16.3, 21.1),
    (200, 9010, 60, 32, 1, 1, 20.1, 33.6, 26.5), (200, 9010, 60, 32, 1, 2, 15.0, 22.2, 20.7),
    (1000, 2998, 3, 2, 1, 2, 11.4, 23.0, 21.4), (1000, 2998, 3, 2, 1, 5, 10.8, 17.8, 18.8),
    (1000, 8964, 19, 8, 1, 1, 21.8, 29.8, 33.3), (2000, 17964, 20, 8, 0, 2, 27.4, 24.7, 55.4),
    (2000, 100652, 75, 32, 1, 1, 88.8, 36.3, 144.2), (4000, 35964, 19, 8, 0, 1, 64.7, 33.3, 119.0),
    (4000, 202776, 75, 32, 1, 10, 48.9, 17.9, 145.1), (400, 1994, 400, 4, 1, 1, 66.2, 46.8, 106.3),
    (4000, 19994, 4000, 4, 0, 5, 449.9, 175.5, 627.7),
]


def test_gmres_choices(rule):
    got = rule([(n, nnz, mr, L, 1024, fp32, m) for n, nnz, mr, L, fp32, m, *_ in GMRES])
    assert len(got) == len(GMRES)
    for case, (_, inside, _) in zip(GMRES, got):
        slot, multi, before = case[6:]
        took = slot if inside else multi
        assert took <= 1.25 * min(slot, multi) and took <= 1.05 * before, case


def test_extremes(rule):
    got = rule([(8192, 8192 * 8192, 8192, 64, 1024, 0, 0), (1, 1, 1, 1, 1024, 0, 0),
                (1, 1, 1, 2, 256, 1, 0), (5, 0, 0, 2, 1024, 0, 0),
                (8000, 39994, 8000, 16, 1024, 0, 0), (8000, 39994, 8000, 64, 1024, 1, 0)])
    assert got[0][1:] == (0, 0)              # a dense matrix: never in one workgroup
    assert got[1] == (1, 1, 1)
    assert got[2][1:] == (1, 1) and got[3][1:] == (1, 1)
    assert got[4][0] == 0 and got[5][0] == 0   # one row of n: the lanes share it
