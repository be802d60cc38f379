// Parameter covariance at a fit: the inverse of the Gauss-Newton Hessian J^T W J of each
// sub-problem (§2.5: the inverse of the Hessian that the LM approximates gives the
// parameter uncertainties and their full covariance).  FP64 throughout.
//
// Sub-problems of at most SMALL_N parameters: one wave factors the block, one row per lane in
// registers, and every lane solves A x = e_c for its own column c, in registers up to 24
// parameters, 8 rows at a time above.  Larger ones:
// the blocked Cholesky of the LM (no damping), then the inverse block column by block column
// -- workgroup j solves L Y = E_j and L^T X = Y for the CHOL_NB columns of block j, with the
// off-diagonal products on FP64 MFMA and the triangular 64 x 64 solves 16 rows at a time, one
// column per lane.  A matrix that is not positive definite yields NaN in its whole block.
//
// Factor mode (the mass-matrix factor of the sampler): only the forward solves, Y = L^{-1},
// stored transposed, F = L^{-T}, so that F F^T = L^{-T} L^{-1} = A^{-1}.
#include "chol_rows.h"

namespace apx {

// Bound by its serial chains.  With the factor and the columns in LDS every step of a solve
// waits for a read and a write; in registers (lane i holds row i of the factor, then lane j
// column j of the inverse) only for the previous step's FMA.
template <int N>
__device__ __forceinline__ void cov_small_n(const Plan& p, const DSub& sb, double* __restrict__ out, int factor, double* L) {
    const int n = sb.n, c = threadIdx.x;
    constexpr int LD = N + 1;
    double* inv = L + N * LD;                        // reciprocals of the diagonal
    {
        double a[N], diag;
        if (!chol_rows<N>(p.A + sb.a_off, n, 0.0, 0.0, a, diag)) {
            if (c < n)
                for (int i = 0; i < n; ++i) out[(long long)i * n + c] = __builtin_nan("");
            return;
        }
        if (c < N) {
#pragma unroll
            for (int j = 0; j < N; ++j) L[c * LD + j] = a[j];
            inv[c] = 1.0 / diag;
        }
    }
    __syncthreads();
    // column c of L^{-1} (zero above row c), then of L^{-T} L^{-1}
    double x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = i == c ? 1.0 : 0.0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        x[m] *= inv[m];
#pragma unroll
        for (int i = m + 1; i < N; ++i) x[i] = fma(-L[i * LD + m], x[m], x[i]);
        if (m % 4 == 3) __builtin_amdgcn_sched_barrier(0);       // keeps the reads of L near their use
    }
    if (!factor) {
#pragma unroll
        for (int m = N - 1; m >= 0; --m) {
            x[m] *= inv[m];
#pragma unroll
            for (int i = 0; i < m; ++i) x[i] = fma(-L[m * LD + i], x[m], x[i]);
            if (m % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (c < n) {
        // row c of F = L^{-T}, or column c of the inverse
        const long long step = factor ? 1 : n, base = factor ? (long long)c * n : c;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (i < n) out[base + i * step] = x[i];
    }
}

// 25 .. SMALL_N parameters: the column lies in LDS and goes through registers in panels of 8 rows
// (with all of it in registers the two solves unroll to thousands of FMAs, over 2000 spilled SGPRs
// and ten minutes to compile: 34 us for 40 parameters, 94 for 41, 96 for 64; now 38, 56, 77; with the
// factor in LDS as well, a row per step, 100, 104, 208).
template <int N>
__device__ __forceinline__ void cov_panels_n(const Plan& p, const DSub& sb, double* __restrict__ out, int factor, double* L) {
    const int n = sb.n, c = threadIdx.x;
    constexpr int LD = N + 2, LY = 65, W = 8;        // LD: rows of whole 16-byte chunks, an odd number of them
    static_assert(N % W == 0, "whole panels");
    double* inv = L + N * LD;                        // reciprocals of the diagonal
    double* Y = inv + N + c;                         // this lane's column, pitch LY
    {
        double a[N], diag;
        if (!chol_rows<N>(p.A + sb.a_off, n, 0.0, 0.0, a, diag)) {
            if (c < n)
                for (int i = 0; i < n; ++i) out[(long long)i * n + c] = __builtin_nan("");
            return;
        }
        if (c < N) {
#pragma unroll
            for (int j = 0; j < N; ++j) L[c * LD + j] = a[j];
            inv[c] = 1.0 / diag;
        }
    }
    const int np = (n + W - 1) / W;                  // rows n .. W np - 1 are identity rows of the factor
    for (int i = 0; i < W * np; ++i) Y[i * LY] = i == c ? 1.0 : 0.0;
    __syncthreads();
    for (int pp = 0; pp < np; ++pp) {                // L y = e_c
        const int r0 = W * pp;
        double x[W];
#pragma unroll
        for (int q = 0; q < W; ++q) x[q] = Y[(r0 + q) * LY];
#pragma unroll
        for (int j = 0; j < W; ++j) {
            x[j] *= inv[r0 + j];
#pragma unroll
            for (int q = j + 1; q < W; ++q) x[q] = fma(-L[(r0 + q) * LD + r0 + j], x[j], x[q]);
        }
#pragma unroll
        for (int q = 0; q < W; ++q) Y[(r0 + q) * LY] = x[q];
#pragma unroll 4
        for (int i = r0 + W; i < n; ++i) {
            double t = Y[i * LY];
#pragma unroll
            for (int q = 0; q < W; ++q) t = fma(-L[i * LD + r0 + q], x[q], t);
            Y[i * LY] = t;
        }
    }
    for (int pp = factor ? -1 : np - 1; pp >= 0; --pp) {     // L^T x = y
        const int r0 = W * pp;
        double x[W];
#pragma unroll
        for (int q = 0; q < W; ++q) x[q] = Y[(r0 + q) * LY];
#pragma unroll
        for (int j = W - 1; j >= 0; --j) {
            x[j] *= inv[r0 + j];
#pragma unroll
            for (int q = 0; q < j; ++q) x[q] = fma(-L[(r0 + j) * LD + r0 + q], x[j], x[q]);
        }
#pragma unroll
        for (int q = 0; q < W; ++q) Y[(r0 + q) * LY] = x[q];
#pragma unroll 4
        for (int i = 0; i < r0; ++i) {
            double t = Y[i * LY];
#pragma unroll
            for (int q = 0; q < W; ++q) t = fma(-L[(r0 + q) * LD + i], x[q], t);
            Y[i * LY] = t;
        }
    }
    if (c < n) {
        // row c of F = L^{-T}, or column c of the inverse
        const long long step = factor ? 1 : n, base = factor ? (long long)c * n : c;
        for (int i = 0; i < n; ++i) out[base + i * step] = Y[i * LY];
    }
}

// Doubles of LDS of a launch for sub-problems of up to N parameters.
constexpr int cov_lds(int N) { return N <= 24 ? N * (N + 2) : N * (N + 2) + N + N * 65; }

template <int NMAX>
__global__ __launch_bounds__(64) void k_cov_small(Plan p, const int* __restrict__ small_subs,
                                                  double* __restrict__ cov, int factor) {
    extern __shared__ double sm[];
    const DSub sb = p.subs[small_subs[blockIdx.x]];
    double* out = cov + sb.a_off;
    if (sb.n == 0) return;
    if (sb.n <= 8) return cov_small_n<8>(p, sb, out, factor, sm);
    if constexpr (NMAX > 8)
        if (sb.n <= 16) return cov_small_n<16>(p, sb, out, factor, sm);
    if constexpr (NMAX > 16)
        if (sb.n <= 24) return cov_small_n<24>(p, sb, out, factor, sm);
    if constexpr (NMAX > 24)
        if (sb.n <= 40) return cov_panels_n<40>(p, sb, out, factor, sm);
    if constexpr (NMAX > 40) cov_panels_n<64>(p, sb, out, factor, sm);
}

hipError_t launch_cov_small(const Plan& p, const int* small_subs, int n_small, int nmax, double* cov,
                            int factor, hipStream_t st) {
    if (n_small <= 0 || nmax <= 0) return hipSuccess;
#define APX_CS(N)                                                                                              \
    hipLaunchKernelGGL(k_cov_small<N>, dim3(n_small), dim3(64), cov_lds(N) * sizeof(double), st, p, \
                       small_subs, cov, factor)
    if (nmax <= 8) APX_CS(8);
    else if (nmax <= 16) APX_CS(16);
    else if (nmax <= 24) APX_CS(24);
    else if (nmax <= 40) APX_CS(40);
    else APX_CS(64);
#undef APX_CS
    return hipGetLastError();
}

// M = A for the undamped factorisation.
__global__ void k_cov_fill(Plan p, int s) {
    const DSub sb = p.subs[s];
    const long long nn = (long long)sb.n * sb.n;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < nn;
         e += (long long)gridDim.x * blockDim.x)
        p.M[sb.a_off + e] = p.A[sb.a_off + e];
}

typedef double cov_d4 __attribute__((ext_vector_type(4)));

// Stage the nr x nc block at (r0, c0) of an n-column row-major matrix into LDS (zeros
// outside), all loads of a thread before its stores.
__device__ __forceinline__ void cov_stage(const double* G, long long ldg, int r0, int c0, int nr, int nc,
                                          double (*B)[CHOL_NB + 1]) {
    constexpr int PER = CHOL_NB * CHOL_NB / 256;
    double v[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = threadIdx.x + 256 * q, i = e >> 6, j = e & 63;
        v[q] = (i < nr && j < nc) ? G[(long long)(r0 + i) * ldg + c0 + j] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = threadIdx.x + 256 * q;
        B[e >> 6][e & 63] = v[q];
    }
}

// T -= op(Lb) * Yb over the 64 x 64 blocks in LDS, T accumulated in acc (each wave a
// 32 x 32 quadrant as 2 x 2 MFMA tiles).  op = identity (forward) or transpose (backward).
template <bool TRANS>
__device__ __forceinline__ void cov_gemm(const double (*Lb)[CHOL_NB + 1], const double (*Yb)[CHOL_NB + 1],
                                         cov_d4 (&acc)[2][2], int lane, int wr, int wc) {
#pragma unroll
    for (int k0 = 0; k0 < CHOL_NB; k0 += 4) {
        double a[2], b[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int row = wr * 32 + m * 16 + (lane & 15), kk = k0 + (lane >> 4);
            a[m] = TRANS ? Lb[kk][row] : Lb[row][kk];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) b[q] = Yb[k0 + (lane >> 4)][wc * 32 + q * 16 + (lane & 15)];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[m][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], b[q], acc[m][q], 0, 0, 0);
    }
}

// Solve L X = T (or L^T X = T with TRANS) in place for the 64 right-hand sides in T, L in Lb
// (nr rows, the rest of Lb zero), the whole workgroup: per 16-row panel, wave 0 takes one
// right-hand side per lane in registers (the panel's entries of L are uniform reads), then the
// rows still to come are updated with the panel on FP64 MFMA by the four waves.  With a row at
// a time in LDS, one wave, the inverse of 99 parameters (two blocks) took 293 us, now 44.
template <bool TRANS>
__device__ __forceinline__ void cov_tri_solve(const double (*Lb)[CHOL_NB + 1], double (*T)[CHOL_NB + 1],
                                              double* invd, int nr) {
    constexpr int W = 16, NP = CHOL_NB / W;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (t < CHOL_NB) invd[t] = t < nr ? 1.0 / Lb[t][t] : 0.0;
    __syncthreads();
    for (int pp = 0; pp < NP; ++pp) {
        const int r0 = W * (TRANS ? NP - 1 - pp : pp);
        if (r0 >= nr) continue;                      // uniform: rows of padding
        if (wv == 0) {
            double x[W];
#pragma unroll
            for (int q = 0; q < W; ++q) x[q] = T[r0 + q][lane];
#pragma unroll
            for (int jj = 0; jj < W; ++jj) {
                const int j = TRANS ? W - 1 - jj : jj;
                x[j] *= invd[r0 + j];
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    if (TRANS ? q < j : q > j)
                        x[q] = fma(-(TRANS ? Lb[r0 + j][r0 + q] : Lb[r0 + q][r0 + j]), x[j], x[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < W; ++q) T[r0 + q][lane] = x[q];
        }
        __syncthreads();
        // T[rows to come] -= L[rows to come, panel] X[panel] (L^T: the panel's rows, transposed)
        const int first = TRANS ? 0 : r0 / W + 1, last = TRANS ? r0 / W : NP;
        for (int e = wv; e < (last - first) * NP; e += 4) {
            const int bi = first + e / NP, bc = e % NP;
            cov_d4 acc = (cov_d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k0 = 0; k0 < W; k0 += 4) {
                const int kk = r0 + k0 + (lane >> 4), row = W * bi + (lane & 15);
                const double a = TRANS ? Lb[kk][row] : Lb[row][kk];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, T[kk][W * bc + (lane & 15)], acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) T[W * bi + (lane >> 4) + 4 * v][W * bc + (lane & 15)] -= acc[v];
        }
        __syncthreads();
    }
}

// Workgroup j: block column j of A^{-1}.  Forward L Y = E_j over row blocks b >= j (Y is
// zero above block j), then backward L^T X = Y over every row block from the last; Y and
// then X live in the output block column.
__global__ __launch_bounds__(256) void k_cov_cols(Plan p, int s, double* __restrict__ cov, int forward_only) {
    __shared__ double Lb[CHOL_NB][CHOL_NB + 1];
    __shared__ double Yb[CHOL_NB][CHOL_NB + 1];
    __shared__ double T[CHOL_NB][CHOL_NB + 1];
    __shared__ double invd[CHOL_NB];
    const DSub sb = p.subs[s];
    const int n = sb.n, nblk = (n + CHOL_NB - 1) / CHOL_NB;
    const int j = blockIdx.x, c0 = j * CHOL_NB, ncl = min(CHOL_NB, n - c0);
    const double* L = p.M + sb.a_off;
    double* X = cov + sb.a_off;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, wr = wv >> 1, wc = wv & 1;
    if (p.lmf[s].chol_fail) {
        for (long long e = t; e < (long long)n * ncl; e += 256) {
            const long long i = e / ncl;
            X[i * n + c0 + (e - i * ncl)] = __builtin_nan("");
        }
        return;
    }
    auto write_T = [&](const cov_d4 (&acc)[2][2]) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    T[wr * 32 + m * 16 + (lane >> 4) + 4 * v][wc * 32 + q * 16 + (lane & 15)] -= acc[m][q][v];
    };
    for (int dir = 0; dir < (forward_only ? 1 : 2); ++dir) {
        const int b_first = dir == 0 ? j : nblk - 1, b_last = dir == 0 ? nblk : -1, step = dir == 0 ? 1 : -1;
        for (int b = b_first; b != b_last; b += step) {
            const int r0 = b * CHOL_NB, nr = min(CHOL_NB, n - r0);
            // T = right-hand side of this block: E_j (forward) or Y (backward)
            if (dir == 0) {
                for (int e = t; e < CHOL_NB * CHOL_NB; e += 256) {
                    const int i = e >> 6, c = e & 63;
                    T[i][c] = (b == j && i == c) ? 1.0 : 0.0;
                }
            } else {
                cov_stage(X, n, r0, c0, nr, ncl, T);
            }
            __syncthreads();
            // minus the products with the blocks already solved
            cov_d4 acc[2][2];
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int q = 0; q < 2; ++q) acc[m][q] = (cov_d4){0.0, 0.0, 0.0, 0.0};
            const int k_first = dir == 0 ? j : b + 1, k_last = dir == 0 ? b : nblk;
            for (int k = k_first; k < k_last; ++k) {
                const int rk = k * CHOL_NB, nk = min(CHOL_NB, n - rk);
                if (dir == 0) cov_stage(L, n, r0, rk, nr, nk, Lb);    // L_bk
                else cov_stage(L, n, rk, r0, nk, nr, Lb);             // L_kb (used transposed)
                cov_stage(X, n, rk, c0, nk, ncl, Yb);
                __syncthreads();
                if (dir == 0) cov_gemm<false>(Lb, Yb, acc, lane, wr, wc);
                else cov_gemm<true>(Lb, Yb, acc, lane, wr, wc);
                __syncthreads();
            }
            write_T(acc);
            cov_stage(L, n, r0, r0, nr, nr, Lb);                      // L_bb
            __syncthreads();
            if (dir == 0) cov_tri_solve<false>(Lb, T, invd, nr);
            else cov_tri_solve<true>(Lb, T, invd, nr);
            for (int e = t; e < nr * CHOL_NB; e += 256) {
                const int i = e >> 6, c = e & 63;
                if (c < ncl) X[(long long)(r0 + i) * n + c0 + c] = T[i][c];
            }
            __syncthreads();
        }
        // forward: zero the rows above block j (the lower-triangular inverse is zero there)
        if (dir == 0)
            for (long long e = t; e < (long long)c0 * ncl; e += 256) {
                const long long i = e / ncl;
                X[i * n + c0 + (e - i * ncl)] = 0.0;
            }
        __syncthreads();
        __threadfence_block();
    }
}

hipError_t launch_cov_cols(const Plan& p, int s, int n, double* cov, int forward_only, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cov_cols, dim3((n + CHOL_NB - 1) / CHOL_NB), dim3(256), 0, st, p, s, cov, forward_only);
    return hipGetLastError();
}

// X <- X^T in place for the n x n block of sub-problem s (each pair swapped by one thread).
__global__ void k_cov_transpose(Plan p, int s, double* __restrict__ X) {
    const DSub sb = p.subs[s];
    const long long n = sb.n, nn = n * n;
    double* B = X + sb.a_off;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < nn;
         e += (long long)gridDim.x * blockDim.x) {
        const long long i = e / n, j = e - i * n;
        if (i < j) {
            const double a = B[i * n + j], b = B[j * n + i];
            B[i * n + j] = b;
            B[j * n + i] = a;
        }
    }
}

hipError_t launch_cov_transpose(const Plan& p, int s, int n, double* X, hipStream_t st) {
    const long long nn = (long long)n * n;
    long long fb = (nn + 255) / 256;
    if (fb > 4096) fb = 4096;
    if (fb < 1) return hipSuccess;
    hipLaunchKernelGGL(k_cov_transpose, dim3((unsigned)fb), dim3(256), 0, st, p, s, X);
    return hipGetLastError();
}

hipError_t launch_cov_fill(const Plan& p, int s, int n, hipStream_t st) {
    const long long nn = (long long)n * n;
    long long fb = (nn + 255) / 256;
    if (fb > 4096) fb = 4096;
    if (fb < 1) return hipSuccess;
    hipLaunchKernelGGL(k_cov_fill, dim3((unsigned)fb), dim3(256), 0, st, p, s);
    return hipGetLastError();
}

}  // namespace apx
