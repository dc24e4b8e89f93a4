"""Who stores what of a CG run's scalars (csrc/cgstate.hpp), compiled on the
host with g++ and run as the device does: the waves of one block read the
state one after the other, and what another block's first thread stores in the
same kernel may land between any two of them.  They have to agree on whether
they run, and a breakdown has to be recorded by the end of the iteration."""
import os
import shutil
import subprocess

import pytest

from helpers import ROOT

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include <initializer_list>
#include <limits>
#include "cgstate.hpp"
using namespace ck;
// one iteration as seen by a block of four waves whose reads of `state` are cut
// after `cut` of them by block 0's stores of the r update; returns the outcome
template <typename T>
int iteration(int before, T sigma, int cut, int *agree) {
    CgDev<T> cg{};
    cg.rho = 4;
    cg.alpha = 7;
    cg.state = before;
    cg.go = 1;
    int ran = 0;
    for (int w = 0; w <= 4; ++w) {
        if (w == cut) {
            if (before == RUN)
                cg_store_sigma(&cg, cg.rho, sigma);
            else
                cg.go = 0;
        }
        if (w < 4)
            ran += cg.state == RUN;
    }
    *agree = ran == 0 || ran == 4;
    // the x/p update: every block reads go, rho_prev and alpha only
    if (!cg.go)
        cg_store_no_step(&cg);
    else if (cg.rho_prev != 4 || cg.alpha != 4 / sigma)
        return -1;
    return cg.state;
}
template <typename T>
int run() {
    const T nan = std::numeric_limits<T>::quiet_NaN();
    const T sigmas[] = {2, 0, -1, nan, std::numeric_limits<T>::infinity()};
    int bad = 0;
    for (int before : {(int)RUN, (int)CONVERGED, (int)BREAKDOWN, (int)BUDGET})
        for (T sigma : sigmas)
            for (int cut = 0; cut <= 4; ++cut) {
                int agree = 0;
                const int got = iteration<T>(before, sigma, cut, &agree);
                const int want = before != RUN ? before : sigma > 0 ? (int)RUN : (int)BREAKDOWN;
                if (!agree || got != want) {
                    printf("before %d sigma %g cut %d: agree %d, state %d, not %d\n", before,
                           (double)sigma, cut, agree, got, want);
                    ++bad;
                }
            }
    return bad;
}
int main() { return run<double>() + run<float>() != 0; }
"""


def test_waves_agree_and_breakdowns_are_recorded(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2411_10143_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
