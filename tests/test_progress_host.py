"""The progress word (csrc/progress.hpp), compiled on the host with g++: packing,
numbers that wrap, and the iterations that have run, counted from reports of
cycles whose last issued steps were skipped."""
import os
import shutil
import subprocess

import pytest

from helpers import ROOT

DRIVER = r"""
#include <cstdio>
#include "progress.hpp"
using namespace ck;
static unsigned rnd = 12345;
static int next(int n) { rnd = rnd * 1664525u + 1013904223u; return (int)((rnd >> 8) % (unsigned)n); }
int main() {
    int bad = 0;
    for (unsigned outcome : {(unsigned)kReportRun, (unsigned)kReportStopped, (unsigned)kReportDone})
        for (unsigned seq : {0u, 1u, 0xffffffu, 0x1000000u, 0x1000005u})
            for (unsigned skipped : {0u, 1u, 63u, 64u, 200u}) {
                const Report r = unpack_report(report_word(0.25f, seq, skipped, outcome));
                bad += r.relres != 0.25 || r.seq != (seq & 0xffffffu) ||
                       r.skipped != (skipped & 63u) || r.outcome != outcome;
            }
    bad += !seq_reached(2, 0xffffffu) || seq_reached(0xffffffu, 2) || !seq_reached(7, 7);
    // a run of cycles: steps are issued, some of a cycle's last are skipped, and the
    // host reads some of the reports; far along, the numbers have wrapped
    for (int start : {0, 0xfffff0}) {
        int issued = start, ran = start;
        RunCount count;
        for (int cycle = 0; cycle < 400; ++cycle) {
            const int steps = 1 + next(30), lost = next(5);
            for (int t = 0; t < steps + lost; ++t) {
                ++issued;
                const Report r = unpack_report(report_word(
                    0.5f, (unsigned)issued, (unsigned)(issued - 1 - ran),
                    t < steps ? kReportRun : kReportStopped));
                const int ahead = next(4);   // the host has issued more by then
                if (next(3) != 0)
                    bad += count.before(r, issued + ahead) != ran;
                ran += t < steps;
            }
        }
    }
    printf("%d\n", bad);
    return bad != 0;
}
"""


def test_words_and_counts(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text("#include <initializer_list>\n" + DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2411_10143_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
