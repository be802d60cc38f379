// The LM state transitions of one sub-problem (§2.5), taken by one thread at the end of the
// launch that sums its chi^2.
#pragma once
#include "apx_internal.h"

namespace apx {

__device__ __forceinline__ void lm_init_state(PlanRef p, int s, double chi2, apx_lm_state* lm) {
    apx_lm_state st;
    st.lambda = APX_LM_LAMBDA0;
    st.chi2 = chi2;
    st.chi2_trial = 0.0;
    st.pred = 0.0;
    st.rho = 0.0;
    st.need_jac = 1;
    st.accepted = 0;
    st.n_accept = 0;
    st.n_reject = 0;
    st.n_chol_retry = 0;
    st.status = isfinite(st.chi2) ? APX_OK : APX_E_NONFINITE;
    lm[s] = st;
    p.spec[s].valid = 0;
}

// Gain ratio, accept or reject, lambda; returns whether the trial parameters are accepted.
__device__ __forceinline__ int lm_accept_state(PlanRef p, int s, double c2t, apx_lm_state* lm) {
    apx_lm_state st = lm[s];
    const LMFlags f = p.lmf[s];
    int accept = 0;
    if (!f.chol_done) {
        st.chi2_trial = __builtin_nan("");
        st.rho = __builtin_nan("");
    } else if (f.trial_bad) {
        st.chi2_trial = __builtin_inf();
        st.rho = -__builtin_inf();
        st.lambda = fmin(st.lambda * APX_LM_UP, APX_LM_LAMBDA_MAX);
    } else {
        const double rho = st.pred != 0.0 ? (st.chi2 - c2t) / st.pred : __builtin_nan("");
        st.chi2_trial = c2t;
        st.rho = rho;
        if (rho > APX_LM_EPS4) {
            accept = 1;
            st.chi2 = c2t;
            st.lambda = fmax(st.lambda / APX_LM_DOWN, APX_LM_LAMBDA_MIN);
        } else {
            st.lambda = fmin(st.lambda * APX_LM_UP, APX_LM_LAMBDA_MAX);
        }
    }
    st.accepted = accept;
    st.need_jac = accept;
    if (accept) st.n_accept += 1; else st.n_reject += 1;
    lm[s] = st;
    // a step solved ahead stays usable only after a rejection of a solved trial (same A,
    // lambda raised exactly once)
    if (accept || !f.chol_done) p.spec[s].valid = 0;
    return accept;
}

}  // namespace apx
