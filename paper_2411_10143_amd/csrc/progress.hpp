// Progress reports: one 8-byte word in pinned host memory per solve, stored by
// one thread of an iteration kernel.  The host reads it to stay a few
// iterations ahead of the device and to stop issuing once the device has
// stopped; nothing is copied or waited for.  Compiled for the host too.
//
//   bits 32-63  the relative residual (float)
//   bits  8-31  the number of the iteration as the host counts them, from 1
//   bits  2-7   how many of the iterations before it did not run (GMRES steps
//               issued after their cycle had stopped), modulo 64
//   bits  0-1   the outcome
#pragma once

#include <cstdint>
#include <cstring>

#if defined(__HIPCC__)
#define CK_HD __host__ __device__
#else
#define CK_HD
#endif

namespace ck {

enum : unsigned { kReportRun = 0, kReportStopped = 1, kReportDone = 2 };

CK_HD inline unsigned long long report_word(float relres, unsigned seq, unsigned skipped,
                                            unsigned outcome) {
    unsigned bits;
    memcpy(&bits, &relres, sizeof bits);
    return ((unsigned long long)bits << 32) | ((seq & 0xffffffu) << 8) | ((skipped & 63u) << 2) |
           outcome;
}

struct Report {
    unsigned seq = 0, skipped = 0, outcome = kReportRun;
    double relres = 0;
};

inline Report unpack_report(unsigned long long v) {
    Report r;
    const unsigned hi = (unsigned)(v >> 32);
    float f;
    memcpy(&f, &hi, sizeof f);
    r.relres = f;
    r.seq = (unsigned)(v >> 8) & 0xffffffu;
    r.skipped = (unsigned)(v >> 2) & 63u;
    r.outcome = (unsigned)v & 3u;
    return r;
}

// a >= b for report numbers, which count modulo 2^24
inline bool seq_reached(unsigned a, unsigned b) { return ((a - b) & 0xffffffu) < 0x800000u; }

// The iterations that have run, from the reports of one run in the order read
// (fewer than 64 iterations are skipped between two of them).
struct RunCount {
    int skipped = 0;
    // before iteration r.seq, of which `issued` is at most 2^24 - 1 ahead
    int before(const Report &r, int issued) {
        skipped += (int)((r.skipped - (unsigned)skipped) & 63u);
        return issued - (int)(((unsigned)issued - r.seq) & 0xffffffu) - 1 - skipped;
    }
};

}  // namespace ck
