// Cholesky factorisation of one small matrix by one wave, rows in registers, shared by the
// damped LM solve and the covariance.
#pragma once
#include "apx_internal.h"

namespace apx {

// 1/sqrt(x) for positive normal x: the hardware estimate refined by two Newton steps
// y <- y (3 - x y^2) / 2 (each roughly doubles the correct bits), a short dependent chain
// on the factorisation's critical path.
__device__ __forceinline__ double rsqrt_f64(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x;
    y = y * fma(-hx * y, y, 1.5);
    y = y * fma(-hx * y, y, 1.5);
    return y;
}

// Value of v in lane `src` (a compile-time constant after unrolling), to every lane.
__device__ __forceinline__ double lane_bcast(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

// One row of an n x n matrix per lane in registers (N >= n columns, padded with identity rows),
// with lam D added to the diagonal (the lane's D): a right-looking Cholesky whose pivot and column entries come
// by readlane, so no column step waits for LDS or a barrier.  Square root and quotients are
// the correctly rounded ones: a fit's later steps depend on the last bits of this one (the
// FP32 derivative images are not continuous in theta), so its arithmetic is part of the
// result.  On return a holds the lane's row of L, diag its diagonal entry; false on a
// non-positive or non-finite pivot.
template <int N>
__device__ __forceinline__ bool chol_rows(const double* __restrict__ A, int n, double lam, double D,
                                          double (&a)[N], double& diag) {
    const int i = threadIdx.x;
#pragma unroll
    for (int j = 0; j < N; ++j) a[j] = (i < n && j < n) ? A[(long long)i * n + j] : (i == j ? 1.0 : 0.0);
#pragma unroll
    for (int j = 0; j < N; ++j)
        if (i == j && j < n) a[j] = fma(lam, D, a[j]);
    bool ok = true;
    diag = 1.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        double piv = lane_bcast(a[k], k);
        // a failed pivot is recorded and replaced by 1 so the (discarded) factor stays finite
        if (!(piv > 0.0) || !isfinite(piv)) { ok = false; piv = 1.0; }
        const double d = sqrt(piv);
        const double l = i > k ? a[k] / d : 0.0;
        a[k] = i > k ? l : (i == k ? d : a[k]);
        if (i == k) diag = d;
#pragma unroll
        for (int j = k + 1; j < N; ++j) a[j] = fma(-l, lane_bcast(l, j), a[j]);
    }
    return ok;
}

}  // namespace apx
