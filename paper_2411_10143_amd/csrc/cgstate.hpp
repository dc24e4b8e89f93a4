// The scalars of a CG run on the device and who stores them when.  Compiled
// for the host too.
//
// A wave reads `state` when it starts, so a kernel in which other blocks still
// start must not store it: the waves of one block would disagree on whether
// they run, and some would leave before the others' barriers.
#pragma once

#if defined(__HIPCC__)
#define CK_HD __host__ __device__
#else
#define CK_HD
#endif

namespace ck {

// Run states shared by the solvers
enum : int { RUN = 0, CONVERGED = 1, BREAKDOWN = 2, BUDGET = 3 };

// CG (Hestenes-Stiefel) scalars.  `state` != RUN makes every iteration
// kernel a no-op, so the host may enqueue ahead of convergence.
template <typename T>
struct CgDev {
    T rho;            // r.r of the current residual
    T rho_prev;       // rho as the sigma finish saw it (read by the x/p
                      // update while its block 0 replaces rho)
    T sigma;          // p.Ap
    T alpha, beta;
    double bnorm;     // ||rhs|| of this (inner) solve
    double tol;       // stop when sqrt(rho)/bnorm <= tol
    double relres;    // last sqrt(rho)/bnorm
    int state;
    int iter;         // iterations completed
    int max_iter;
    int go;           // set by the sigma finish: 1 when this iteration's
                      // x/p update runs (state RUN and sigma > 0)
};

// The sigma finish of a running solve: what one thread stores.  The r update
// does this in its block 0 while other blocks of it may not have started, so a
// breakdown (sigma <= 0 or not a number) is left in `go` for the next kernel.
template <typename T>
CK_HD inline void cg_store_sigma(CgDev<T> *cg, T rho, T sigma) {
    const bool ok = sigma > T(0);
    cg->sigma = sigma;
    cg->rho_prev = rho;
    cg->go = ok;
    if (ok)
        cg->alpha = rho / sigma;
}

// The x/p update of an iteration that does not run (`go` is 0), in which no
// block reads `state`: the solve had stopped before, or breaks down here.
template <typename T>
CK_HD inline void cg_store_no_step(CgDev<T> *cg) {
    if (cg->state == RUN)
        cg->state = BREAKDOWN;
}

}  // namespace ck
