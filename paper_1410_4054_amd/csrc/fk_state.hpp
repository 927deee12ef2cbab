// Device-side steps every solver kernel shares: coherent access to words that
// other workgroups read in the same launch, and the scalar work of a
// reduction point (finalize).
#pragma once

#include <hip/hip_runtime.h>

#include "fk_internal.hpp"

namespace fk {
namespace {

// Device-coherent (agent-scope) store and load of one double.
__device__ __forceinline__ void store_coherent(double *p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double load_coherent(const double *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------- finalize

__device__ __forceinline__ void put_hist(const DevState *st, double *hist, int it, double v)
{
    if (hist && it < st->hist_cap)
        hist[it] = v;
}

__device__ __forceinline__ void put_scal(const DevState *st, double *scal, int it, int slot, double v)
{
    if (scal && it < st->hist_cap)
        scal[4 * it + slot] = v;
}

// Scalar work of a reduction point (one thread).  The expressions and their
// order follow Algorithms 1-4 exactly; see the comments per case.
// Algorithm 2, alpha_i = <r_i,r_i> / <p_i,Ap_i> and beta_i by Eq. (3).
__device__ void cg_alpha(DevState *st, double pap, double apap, double *scal)
{
    if (!(pap > 0.0) || !isfinite(pap) || !isfinite(apap)) {
        st->status = ST_BREAKDOWN;
        return;
    }
    const double alpha = st->rr / pap;
    const double beta = alpha * alpha * apap / st->rr - 1.0;  // Eq. (3)
    st->alpha = alpha;
    st->beta = beta;
    put_scal(st, scal, st->it, 0, alpha);
    put_scal(st, scal, st->it, 1, beta);
    if (st->it >= st->max_iter)
        st->status = ST_NOT_CONVERGED;
}

// Algorithm 2, <r_i, r_i>: iteration i done, residual history, convergence.
__device__ void cg_rr(DevState *st, double rr, double *hist, double *scal)
{
    const int it = st->it + 1;
    st->it = it;
    st->rr = rr;
    const double rel = sqrt(rr) / st->bnorm;
    st->last_rel = rel;
    put_hist(st, hist, it, rel);
    put_scal(st, scal, it - 1, 3, rr);
    if (!isfinite(rr))
        st->status = ST_BREAKDOWN;
    else if (sqrt(rr) <= st->tol)
        st->status = ST_CONVERGED;
    else if (it >= st->max_iter)
        st->status = ST_NOT_CONVERGED;
}

// Algorithm 2 in FP32 (the FP32-accumulating inner solver): the same steps
// with alpha_i, beta_i (Eq. (3)), the norm and the test formed in FP32.
// The state's doubles hold the FP32 values exactly.
__device__ void cg_alpha32(DevState *st, float pap, float apap)
{
    if (!(pap > 0.0f) || !isfinite(pap) || !isfinite(apap)) {
        st->status = ST_BREAKDOWN;
        return;
    }
    const float rr = (float)st->rr;
    const float alpha = rr / pap;
    const float beta = alpha * alpha * apap / rr - 1.0f;  // Eq. (3)
    st->alpha = alpha;
    st->beta = beta;
    if (st->it >= st->max_iter)
        st->status = ST_NOT_CONVERGED;
}

__device__ void cg_rr32(DevState *st, float rr)
{
    const int it = st->it + 1;
    st->it = it;
    st->rr = rr;
    st->last_rel = (double)sqrtf(rr) / st->bnorm;
    if (!isfinite(rr))
        st->status = ST_BREAKDOWN;
    else if (sqrtf(rr) <= (float)st->tol)
        st->status = ST_CONVERGED;
    else if (it >= st->max_iter)
        st->status = ST_NOT_CONVERGED;
}

// Algorithm 4: omega_i = <As,s>/<As,As>, beta_i = -<As,r0*>/<Ap,r0*> (the
// form of Section 3.2), and <r_{i+1}, r_{i+1}> expanded in <s,s>, <s,As>,
// <As,As>.
// Algorithms 3/4: alpha_i = rho_i / <Ap_i, r0*>.
__device__ void b_alpha(DevState *st, double apr, double *scal)
{
    const double rho = st->rho;
    if (apr == 0.0 || !isfinite(apr) || rho == 0.0 || !isfinite(rho)) {
        st->status = ST_BREAKDOWN;
        return;
    }
    st->apr = apr;
    st->alpha = rho / apr;
    put_scal(st, scal, st->it, 0, st->alpha);
}

__device__ void b_omega(DevState *st, double ass, double asas, double asr, double *scal)
{
    if (asas == 0.0 || !isfinite(asas) || !isfinite(ass) || !isfinite(asr)) {
        st->status = ST_BREAKDOWN;
        return;
    }
    const double beta = -asr / st->apr;  // via <s_i, r0*> = 0
    const double omega = ass / asas;
    st->beta = beta;
    st->omega = omega;
    st->rr_next = st->ss - 2.0 * omega * ass + omega * omega * asas;
    put_scal(st, scal, st->it, 1, beta);
    put_scal(st, scal, st->it, 2, omega);
}

__device__ void finalize(DevState *st, int fin, const double *d, int K, double *hist, double *scal)
{
    for (int k = 0; k < K; ++k)
        st->dots[k] = d[k];
    switch (fin) {
    case FIN_NONE:
        break;
    case FIN_SETUP: {  // d = {<r0,r0>, <b,b>}
        const double rr = d[0], bb = d[1];
        st->it = 0;
        st->rho_pub = 0;
        st->rr = rr;
        st->rho = rr;  // r0* = r0, so <r0, r0*> = <r0, r0>
        if (bb == 0.0) {
            st->bnorm = 0.0;
            st->tol = 0.0;
            st->last_rel = 0.0;
            put_hist(st, hist, 0, 0.0);
            st->status = ST_ZERO_RHS;
            break;
        }
        const double bnorm = sqrt(bb);
        st->bnorm = bnorm;
        st->tol = st->rtol * bnorm;
        const double rel = sqrt(rr) / bnorm;
        st->last_rel = rel;
        put_hist(st, hist, 0, rel);
        if (!isfinite(rr))
            st->status = ST_BREAKDOWN;
        else if (sqrt(rr) <= st->tol)
            st->status = ST_CONVERGED;
        break;
    }
    case FIN_CG_ALPHA:  // Algorithm 2: d = {<p_i,Ap_i>, <Ap_i,Ap_i>}
        cg_alpha(st, d[0], d[1], scal);
        break;
    case FIN_SETUP32: {  // FP32 inner start: d = {<r0,r0>, <r0,r0>} (FP32 values)
        const float rr = (float)d[0];
        st->it = 0;
        st->rho_pub = 0;
        st->rr = rr;
        if (rr == 0.0f) {
            st->bnorm = 0.0;
            st->tol = 0.0;
            st->last_rel = 0.0;
            st->status = ST_ZERO_RHS;
            break;
        }
        if (!isfinite(rr)) {
            st->status = ST_BREAKDOWN;
            break;
        }
        const float tol = (float)st->rtol * sqrtf(rr);
        st->bnorm = (double)sqrtf(rr);
        st->tol = tol;
        st->last_rel = 1.0;
        if (sqrtf(rr) <= tol)
            st->status = ST_CONVERGED;
        break;
    }
    case FIN_CG_ALPHA32:  // d = {<p_i,Ap_i>, <Ap_i,Ap_i>} (FP32 values)
        cg_alpha32(st, (float)d[0], (float)d[1]);
        break;
    case FIN_CG_RR_ALPHA32:  // d = {<p_i,Ap_i>, <Ap_i,Ap_i>, <r_i,r_i>} (FP32 values)
        cg_rr32(st, (float)d[2]);
        if (st->status == ST_RUNNING)
            cg_alpha32(st, (float)d[0], (float)d[1]);
        break;
    case FIN_CG_RR:  // Algorithm 2: d = {<r_i,r_i>}
        cg_rr(st, d[0], hist, scal);
        break;
    case FIN_CG_RR_ALPHA:  // d = {<p_i,Ap_i>, <Ap_i,Ap_i>, <r_i,r_i>}
        // The convergence test on r_i comes first, as when <r_i,r_i> is
        // reduced on its own; alpha_i, beta_i only while still running.
        cg_rr(st, d[2], hist, scal);
        if (st->status == ST_RUNNING)
            cg_alpha(st, d[0], d[1], scal);
        break;
    case FIN_B_ALPHA:  // Algorithms 3/4: d = {<Ap_i, r0*>}
        b_alpha(st, d[0], scal);
        break;
    case FIN_B_RHO_ALPHA:  // d = {<Ap_i, r0*>, <r_i, r0*>, <r_i, r_i>}
        // rho_i and the direct <r_i,r_i> come from the update's published
        // partials, except in the first iteration (rho_0 from the setup).
        if (st->rho_pub) {
            st->rho = d[1];
            st->rr = d[2];
            st->rho_pub = 0;
        }
        b_alpha(st, d[0], scal);
        break;
    case FIN_B_XRP_ALPHA:  // d = {<Ap_{i+1}, r0*>, <r_{i+1}, r0*>, <r_{i+1}, r_{i+1}>}
        // (two-kernel schedule: the update and the product in one launch)
        st->rho = d[1];
        st->rr = d[2];
        b_alpha(st, d[0], scal);
        break;
    case FIN_B_SS: {  // d = {<s_i, s_i>}: half-step test
        st->ss = d[0];
        if (sqrt(d[0]) <= st->tol)
            st->status = ST_HALF;
        break;
    }
    case FIN_B_OMEGA:  // Algorithm 4: d = {<As,s>, <As,As>, <As,r0*>}
        b_omega(st, d[0], d[1], d[2], scal);
        break;
    case FIN_B_SS_OMEGA: {  // d = {<As,s>, <As,As>, <As,r0*>, <s,s>}
        // The half-step test on s_i first, as when <s_i,s_i> is reduced on
        // its own; omega, beta only while still running.  The decision on
        // iteration i+1 needs only the expanded <r_{i+1}, r_{i+1}> and omega,
        // so it is taken here; the x, r, p update still runs after it.
        st->ss = d[3];
        if (sqrt(d[3]) <= st->tol) {
            st->status = ST_HALF;
            break;
        }
        b_omega(st, d[0], d[1], d[2], scal);
        if (st->status != ST_RUNNING)
            break;
        const int it = st->it + 1;
        st->it = it;
        const double rr_next = st->rr_next;
        const double rnorm = sqrt(rr_next > 0.0 ? rr_next : 0.0);
        const double rel = rnorm / st->bnorm;
        st->last_rel = rel;
        put_hist(st, hist, it, rel);
        put_scal(st, scal, it - 1, 3, rr_next);
        if (!isfinite(rr_next))
            st->status = ST_FINAL_BREAKDOWN;
        else if (rnorm <= st->tol)
            st->status = ST_FINAL_CONVERGED;
        else if (st->omega == 0.0)
            st->status = ST_FINAL_BREAKDOWN;
        else if (it >= st->max_iter)
            st->status = ST_FINAL_NOT_CONVERGED;
        break;
    }
    case FIN_B_XRP_PUB:  // the update after a decision: d = {<r,r0*>, <r,r>}
        if (st->status == ST_HALF) {
            const int it = st->it + 1;
            st->it = it;
            const double rel = sqrt(st->ss) / st->bnorm;
            st->last_rel = rel;
            put_hist(st, hist, it, rel);
            put_scal(st, scal, it - 1, 3, st->ss);
            st->status = ST_CONVERGED;
            break;
        }
        st->rho = d[0];
        st->rr = d[1];
        st->status = st->status == ST_FINAL_CONVERGED       ? ST_CONVERGED
                     : st->status == ST_FINAL_NOT_CONVERGED ? ST_NOT_CONVERGED
                                                            : ST_BREAKDOWN;
        break;
    case FIN_B_XRP: {  // Algorithm 4: d = {<r_{i+1}, r0*>, <r_{i+1}, r_{i+1}>}
        const int it = st->it + 1;
        st->it = it;
        if (st->status == ST_HALF) {
            const double rel = sqrt(st->ss) / st->bnorm;
            st->last_rel = rel;
            put_hist(st, hist, it, rel);
            put_scal(st, scal, it - 1, 3, st->ss);
            st->status = ST_CONVERGED;
            break;
        }
        st->rho = d[0];
        st->rr = d[1];
        const double rr_next = st->rr_next;
        const double rnorm = sqrt(rr_next > 0.0 ? rr_next : 0.0);
        const double rel = rnorm / st->bnorm;
        st->last_rel = rel;
        put_hist(st, hist, it, rel);
        put_scal(st, scal, it - 1, 3, rr_next);
        if (!isfinite(rr_next))
            st->status = ST_BREAKDOWN;
        else if (rnorm <= st->tol)
            st->status = ST_CONVERGED;
        else if (st->omega == 0.0)
            st->status = ST_BREAKDOWN;
        else if (it >= st->max_iter)
            st->status = ST_NOT_CONVERGED;
        break;
    }
    case FIN_C_CG_ALPHA: {  // Algorithm 1: d = {<p_i, A p_i>}
        const double pq = d[0];
        if (!(pq > 0.0) || !isfinite(pq)) {
            st->status = ST_BREAKDOWN;
            break;
        }
        st->alpha = st->rr / pq;
        put_scal(st, scal, st->it, 0, st->alpha);
        break;
    }
    case FIN_C_CG_BETA: {  // Algorithm 1: d = {<r_{i+1}, r_{i+1}>}
        const double rr_new = d[0];
        const int it = st->it + 1;
        st->it = it;
        const double rel = sqrt(rr_new) / st->bnorm;
        st->last_rel = rel;
        put_hist(st, hist, it, rel);
        put_scal(st, scal, it - 1, 3, rr_new);
        if (!isfinite(rr_new)) {
            st->status = ST_BREAKDOWN;
        } else if (sqrt(rr_new) <= st->tol) {
            st->status = ST_CONVERGED;
        } else if (it >= st->max_iter) {
            st->status = ST_NOT_CONVERGED;
        } else {
            st->beta = rr_new / st->rr;
            put_scal(st, scal, it - 1, 1, st->beta);
            st->rr = rr_new;
        }
        break;
    }
    case FIN_C_B_OMEGA: {  // Algorithm 3: d = {<t,s>, <t,t>}, t = A s_i
        const double ts = d[0], tt = d[1];
        if (tt == 0.0 || !isfinite(tt) || !isfinite(ts)) {
            st->status = ST_BREAKDOWN;
            break;
        }
        st->omega = ts / tt;
        put_scal(st, scal, st->it, 2, st->omega);
        break;
    }
    case FIN_C_B_RR: {  // Algorithm 3: d = {<r_{i+1}, r_{i+1}>}
        const double rr = d[0];
        const int it = st->it + 1;
        st->it = it;
        st->rr = rr;
        const double rel = sqrt(rr) / st->bnorm;
        st->last_rel = rel;
        put_hist(st, hist, it, rel);
        put_scal(st, scal, it - 1, 3, rr);
        if (!isfinite(rr))
            st->status = ST_BREAKDOWN;
        else if (sqrt(rr) <= st->tol)
            st->status = ST_CONVERGED;
        break;
    }
    case FIN_C_B_RHO: {  // Algorithm 3: d = {<r_{i+1}, r0*>}
        const double rho_new = d[0];
        if (st->omega == 0.0 || rho_new == 0.0 || !isfinite(rho_new)) {
            st->status = ST_BREAKDOWN;
            break;
        }
        st->beta = (rho_new / st->rho) * (st->alpha / st->omega);
        put_scal(st, scal, st->it - 1, 1, st->beta);
        st->rho = rho_new;
        if (st->it >= st->max_iter)
            st->status = ST_NOT_CONVERGED;
        break;
    }
    case FIN_MIX_OUTER: {  // mixed precision: d = {<r,r>, <b,b>} of r = b - A x in FP64
        const double rr = d[0], bb = d[1];
        const int it = st->it;  // residuals evaluated so far
        if (it == 0) {
            if (bb == 0.0) {
                st->bnorm = 0.0;
                st->tol = 0.0;
                st->last_rel = 0.0;
                put_hist(st, hist, 0, 0.0);
                st->it = 1;
                st->status = ST_ZERO_RHS;
                break;
            }
            st->bnorm = sqrt(bb);
            st->tol = st->rtol * st->bnorm;
        }
        st->rr = rr;
        const double rel = sqrt(rr) / st->bnorm;
        st->last_rel = rel;
        put_hist(st, hist, it, rel);
        st->it = it + 1;
        if (!isfinite(rr))
            st->status = ST_BREAKDOWN;
        else if (sqrt(rr) <= st->tol)
            st->status = ST_CONVERGED;
        break;
    }
    case FIN_GM_SETUP: {  // GMRES cycle start: d = {<r0,r0>, <b,b>}
        const double rr = d[0], bb = d[1];
        if (st->bnorm == 0.0) {  // first cycle of the solve
            if (bb == 0.0) {
                st->last_rel = 0.0;
                put_hist(st, hist, 0, 0.0);
                st->status = ST_ZERO_RHS;
                break;
            }
            st->bnorm = sqrt(bb);
            st->tol = st->rtol * st->bnorm;
        }
        const double rho0 = sqrt(rr);
        st->rho0 = rho0;
        st->last_rel = rho0 / st->bnorm;
        put_hist(st, hist, st->it, rho0 / st->bnorm);
        if (!isfinite(rho0))
            st->status = ST_BREAKDOWN;
        else if (rho0 <= st->tol)
            st->status = ST_CONVERGED;
        else if (st->it >= st->max_iter)
            st->status = ST_NOT_CONVERGED;
        else {
            st->zeta2 = 1.0;
            st->gi = 1;
        }
        break;
    }
    case FIN_GM_R1:  // R[i-1][i] = <v_{i-1}, w> (scal points to R)
        scal[(st->gi - 1) * (st->gm + 1) + st->gi] = d[0];
        break;
    case FIN_GM_NORM: {  // R[i][i] = ||w||; a zero or non-finite norm ends the cycle before step i
        const double rii = sqrt(d[0]);
        if (!(rii > 0.0) || !isfinite(rii))
            st->status = ST_CYCLE_DONE;
        else
            scal[st->gi * (st->gm + 1) + st->gi] = rii;
        break;
    }
    case FIN_GM_XI: {  // xi_i = <r, v_i>; norm estimate rho0 sqrt(zeta2)
        const double xi = d[0];
        const int i = st->gi;
        scal[i] = xi;  // row 0 of R
        double z = st->zeta2 - xi * xi;
        if (z < 0.0)
            z = 0.0;
        st->zeta2 = z;
        const int it = st->it + 1;
        st->it = it;
        const double est = st->rho0 * sqrt(z);
        st->last_rel = est / st->bnorm;
        put_hist(st, hist, it, est / st->bnorm);
        st->gi = i + 1;
        if (est <= st->tol || i + 1 > st->gm || it >= st->max_iter)
            st->status = ST_CYCLE_DONE;
        break;
    }
    case FIN_HALF_DONE: {  // BiCGStab exit after the half step
        const int it = st->it + 1;
        st->it = it;
        const double rel = sqrt(st->ss) / st->bnorm;
        st->last_rel = rel;
        put_hist(st, hist, it, rel);
        put_scal(st, scal, it - 1, 3, st->ss);
        st->status = ST_CONVERGED;
        break;
    }
    default:
        break;
    }
}

}  // namespace
}  // namespace fk
