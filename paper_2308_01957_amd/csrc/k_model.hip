// Component evaluation kernels: parameter preparation (b_n on the device), the
// supersampled pre-convolution render, derivative images for the Jacobian and the
// adjoint contraction for the chi^2 gradient.
//
// Profile (Sersic, §2.1.1): I(R) = Ie exp(-b_n ((R/Re)^(1/n) - 1)) with elliptical
// R = sqrt(x'^2 + (y'/q)^2), x' = dx cos PA + dy sin PA, y' = -dx sin PA + dy cos PA.
// It is evaluated as I = 2^(A - B t), t = 2^(g log2 R^2 - h) with A = log2 Ie + b log2 e,
// B = b log2 e, g = 1/(2n), h = log2(Re)/n: three hardware transcendentals (v_log_f32,
// v_exp_f32) per sub-pixel node, the exponent arithmetic in FP64 (full rate on CDNA4)
// so the FP32 result carries only the transcendentals' rounding.
// Pixel integration (§2.1.2): area * sum_k w_k I(node_k) over s x s nodes.
#include "apx_internal.h"
#include "sersic64.h"

namespace apx {

#define LN2F 0.69314718055994531f
#define LN10F 2.3025850929940457f

// ------------------------------------------------------------------------ b_n
// b_n and db_n/dn by cubic Hermite interpolation of the host-built FP64 table (nodes
// every 1/256 in n; interpolation error below 1e-10 relative on [0.36, 10]).
__device__ void sersic_bn_table(const double* tab, double n, double& b, double& bp) {
    const double u = (n - BN_N0) * BN_INV_H;
    int k = (int)floor(u);
    k = k < 0 ? 0 : (k > BN_COUNT - 2 ? BN_COUNT - 2 : k);
    const double t = u - k, h = 1.0 / BN_INV_H;
    const double b0 = tab[2 * k], d0 = tab[2 * k + 1], b1 = tab[2 * k + 2], d1 = tab[2 * k + 3];
    const double t2 = t * t, t3 = t2 * t;
    b = (2 * t3 - 3 * t2 + 1) * b0 + (t3 - 2 * t2 + t) * h * d0 + (-2 * t3 + 3 * t2) * b1 + (t3 - t2) * h * d1;
    bp = (6 * t2 - 6 * t) * BN_INV_H * b0 + (3 * t2 - 4 * t + 1) * d0 + (-6 * t2 + 6 * t) * BN_INV_H * b1 +
         (3 * t2 - 2 * t) * d1;
}

// ------------------------------------------------------------------- re-centring taps
// Weights that move a pixel-sampled image by delta (|delta| <= 1/2) along one axis,
// shifted(i) = sum_t w[t + a] img(i - t), and their derivatives in delta (§2.1.3).
// Bilinear: the two nearest samples (derivative from the right at delta = 0).  Lanczos of
// order a: sinc(t - delta) sinc((t - delta) / a) (normalised sinc), divided by its sum.
__device__ __forceinline__ double nsinc(double x) { return x == 0.0 ? 1.0 : sinpi(x) / (M_PI * x); }
__device__ __forceinline__ double nsinc_d(double x) { return x == 0.0 ? 0.0 : (cospi(x) - nsinc(x)) / x; }

__device__ void shift_taps(int method, int a, double delta, double* w, double* dw) {
    if (method == APX_SHIFT_BILINEAR) {
        const double side = delta >= 0.0 ? 1.0 : -1.0;
        for (int j = 0; j < 3; ++j) {
            const double t = (double)(j - 1);
            w[j] = fmax(0.0, 1.0 - fabs(t - delta));
            dw[j] = (t == 0.0 ? -side : 0.0) + (t == side ? side : 0.0);
        }
        return;
    }
    double N = 0.0, dN = 0.0;
    for (int j = 0; j <= 2 * a; ++j) {
        const double x = (double)(j - a) - delta;
        const bool in = fabs(x) < (double)a;
        const double L = in ? nsinc(x) * nsinc(x / a) : 0.0;
        const double dL = in ? -(nsinc_d(x) * nsinc(x / a) + nsinc(x) * nsinc_d(x / a) / a) : 0.0;
        w[j] = L;
        dw[j] = dL;
        N += L;
        dN += dL;
    }
    for (int j = 0; j <= 2 * a; ++j) {
        dw[j] = (dw[j] * N - w[j] * dN) / (N * N);
        w[j] = w[j] / N;
    }
}

// ------------------------------------------------------------------------- prep
// The start of every evaluation in one launch: component constants and skies, stamps, and, in
// an LM iteration, what precedes them (the iteration's flags and adopted steps, or the trial
// parameters theta + h).  These are a handful of microseconds of work each, and as launches
// of their own they cost a small fit more than the work (a 64 x 64 fit spent 20 launches an
// iteration, 98 us of which 65 were kernels).  Block ranges, in order: components and images;
// one block per image's stamp; the begin blocks; the trial parameters.
struct PrepBlocks { int comps, psf, begin, trial; };

// theta[k] of the evaluation: the caller's, or with a step theta + h where the solve succeeded
__device__ __forceinline__ double prep_theta(PlanRef p, const PrepIO& io, int k) {
    double v = io.theta[k];
    if (io.step) {
        const int s = p.par_sub[k];
        if (s >= 0 && p.lmf[s].chol_done) v += io.step[k];
    }
    return v;
}

// Start of an iteration: clear the per-iteration flags of both solve copies and decide
// whether a large sub-problem takes the step solved ahead: the same A (its last trial was
// rejected, so no new normal equations) and the lambda that solve started from.
__device__ __forceinline__ int lm_begin_sub(PlanRef p, const apx_lm_state* lm, int s) {
    LMFlags f;
    f.chol_done = 0;
    f.chol_fail = 0;
    f.trial_bad = 0;
    f.skip = 0;
    f.subst_fail = 0;
    f.rhs_folded = 0;
    f.adopted = 0;
    p.lmf[p.n_sub + s] = f;
    const LMSpec sp = p.spec[s];
    f.adopted = p.subs[s].large && sp.valid && lm[s].need_jac == 0 && lm[s].lambda == sp.lam_start;
    p.lmf[s] = f;
    return f.adopted;
}

// One wave per sub-problem (problems with a large sub-problem, whose solves are made ahead):
// an adopting sub-problem takes the step, its predicted decrease, lambda and retry count from
// the solve made ahead (exactly what solving now would give: same A, D, g and starting
// lambda, same kernels), and the record is used up.
__device__ __forceinline__ void lm_adopt_sub(PlanRef p, apx_lm_state* lm, int s) {
    if (threadIdx.x >= 64) return;
    int adopted = 0;
    if (threadIdx.x == 0) adopted = lm_begin_sub(p, lm, s);
    adopted = __shfl(adopted, 0, 64);
    if (!adopted) return;
    const DSub sb = p.subs[s];
    for (int i = (int)threadIdx.x; i < sb.n; i += 64) p.hvec[sb.p0 + i] = p.hvec[p.n_par + sb.p0 + i];
    if (threadIdx.x == 0) {
        const LMSpec sp = p.spec[s];
        lm[s].pred = sp.pred;
        lm[s].lambda = sp.lam_final;
        lm[s].n_chol_retry += sp.retries;
        p.lmf[s].chol_done = sp.done;
        p.spec[s].valid = 0;
    }
}

__device__ void prep_comp(PlanRef p, const PrepIO& io, int i) {
    const int lm_trial = io.mark;
    if (i < p.n_images) {
        const DImage& im = p.images[i];
        const double sky = im.sky_par >= 0 ? prep_theta(p, io, im.sky_par) : im.sky_fixed;
        p.sky_val[i] = sky;
        if (!isfinite(sky)) {
            if (lm_trial) atomicOr(&p.lmf[im.sub].trial_bad, 1);
            else atomicOr(p.sticky, FLAG_NONFINITE);
        }
    }
    if (i >= p.n_comps) return;
    const DComp cp = p.comps[i];
    const DImage& im = p.images[cp.image];
    double v[7];
    bool finite = true;
    for (int k = 0; k < 7; ++k) {
        v[k] = cp.par[k] >= 0 ? prep_theta(p, io, cp.par[k]) : cp.fixed[k];
        finite = finite && isfinite(v[k]);
    }
    CompConst c;
    c.x0 = c.y0 = c.cs_d = c.sn_d = c.q_d = c.iq_d = c.kre = c.h_d = c.A_d = c.B_d = c.g_d = 0.0;
    c.ax = c.ay = c.bx = c.by = c.qxx = c.qxy = c.qyy = c.qmax = 0.0;
    for (int k = 0; k < BIN_DEG; ++k) c.bin[k] = 0.0;
    c.cs = c.sn = c.iq = c.g = c.b = c.bp = c.n = c.re = c.q = c.F = 0.f;
    c.pad = 0;
    c.F64 = 0.0;
    bool valid = finite;
    if (cp.type == APX_SERSIC) {
        const double q = v[2], pa = v[3], n = v[4], re = v[5], lie = v[6];
        valid = valid && q >= 0.01 && q <= 1.0 && n >= 0.36 && n <= 10.0 && re >= 0.01 && re <= 1e4;
        if (valid) {
            double b, bp;
            sersic_bn_table(p.bn_tab, n, b, bp);
            const double log2e = 1.4426950408889634;
            c.x0 = v[0];
            c.y0 = v[1];
            c.cs_d = cos(pa);
            c.sn_d = sin(pa);
            c.q_d = q;
            c.iq_d = 1.0 / q;
            c.kre = p.k_re * re;
            c.h_d = log2(re) / n;
            c.A_d = lie * 3.3219280948873622 + b * log2e;
            c.B_d = b * log2e;
            c.g_d = 0.5 / n;
            c.ax = fma(im.aff[1], c.cs_d, im.aff[4] * c.sn_d);
            c.bx = fma(im.aff[2], c.cs_d, im.aff[5] * c.sn_d);
            c.ay = fma(im.aff[4], c.cs_d, -(im.aff[1] * c.sn_d)) * c.iq_d;
            c.by = fma(im.aff[5], c.cs_d, -(im.aff[2] * c.sn_d)) * c.iq_d;
            c.qxx = c.ax * c.ax + c.ay * c.ay;
            c.qxy = 2.0 * (c.ax * c.bx + c.ay * c.by);
            c.qyy = c.bx * c.bx + c.by * c.by;
            c.qmax = (c.qxx + fabs(c.qxy) + c.qyy) * p.node_max * p.node_max;
            c.bin[0] = c.g_d;
#pragma unroll
            for (int k = 1; k < BIN_DEG; ++k) c.bin[k] = c.bin[k - 1] * (c.g_d - k) * (1.0 / (k + 1));
            c.cs = (float)c.cs_d;
            c.sn = (float)c.sn_d;
            c.iq = (float)(1.0 / q);
            c.g = (float)(0.5 / n);
            c.b = (float)b;
            c.bp = (float)bp;
            c.n = (float)n;
            c.re = (float)re;
            c.q = (float)q;
            if (p.shift != APX_SHIFT_NONE) {
                // sample with the centre at the nearest pixel centre n; the taps move the
                // result back by delta = (pixel position) - n
                const double px = im.inv[0] + im.inv[1] * c.x0 + im.inv[2] * c.y0;
                const double py = im.inv[3] + im.inv[4] * c.x0 + im.inv[5] * c.y0;
                const double nx = floor(px + 0.5), ny = floor(py + 0.5);
                c.x0 = im.aff[0] + im.aff[1] * nx + im.aff[2] * ny;
                c.y0 = im.aff[3] + im.aff[4] * nx + im.aff[5] * ny;
                double* tp = p.stap + (long long)i * STAP_STRIDE;
                shift_taps(p.shift, p.shift_a, px - nx, tp, tp + 2 * SHIFT_NT);
                shift_taps(p.shift, p.shift_a, py - ny, tp + SHIFT_NT, tp + 3 * SHIFT_NT);
            }
        }
    } else {
        // point source: sky position -> pixel position of its image
        const double ux = v[0], uy = v[1];
        const double px = im.inv[0] + im.inv[1] * ux + im.inv[2] * uy;
        const double py = im.inv[3] + im.inv[4] * ux + im.inv[5] * uy;
        c.x0 = px;
        c.y0 = py;
        c.F64 = exp(v[2] * 2.302585092994046);
        c.F = (float)c.F64;
    }
    c.valid = valid ? 1 : 0;
    if (cp.type == APX_SERSIC && p.shift != APX_SHIFT_NONE && !valid)
        for (int j = 0; j < STAP_STRIDE; ++j) p.stap[(long long)i * STAP_STRIDE + j] = 0.0;
    p.cc[i] = c;
    if (!valid) {
        if (lm_trial) atomicOr(&p.lmf[cp.sub].trial_bad, 1);
        else atomicOr(p.sticky, FLAG_DOMAIN);
    }
}

// Stamps of every image for this theta: fixed stamps promoted to FP64 (objective
// convolution); live Moffat stamps (§2.1.3, §3.4) rendered at the integer offsets,
// normalised, with d/dn and d/dR_d of the normalised stamp (quotient rule), in FP64 and
// as FP32 copies for the FP32 kernels; with io.flip, the flipped stamps of the adjoint.  One
// workgroup per image; the sums are ordered.
__device__ void prep_psf(PlanRef p, const PrepIO& io, int k) {
    __shared__ double red[4][3];
    const int lm_trial = io.mark;
    const DImage& im = p.images[k];
    const int P = im.P, c = im.c, P2 = P * P;
    double* K64 = p.psf64 + im.psf_off;
    if (!im.live) {
        const float* K = p.psf + im.psf_off;
        int sym = 1;
        for (int e = threadIdx.x; e < P2; e += blockDim.x) {
            const int u = e / P;
            K64[e] = (double)K[e];
            sym &= K[e] == K[e + (P - 1 - 2 * u) * P];   // false for a NaN: then no rows are paired
            if (io.flip) p.psf_flip[im.psf_off + P2 - 1 - e] = K[e];
        }
        sym = __syncthreads_and(sym);
        if (threadIdx.x == 0) p.psf_sym[k] = sym;
        return;
    }
    if (threadIdx.x == 0) p.psf_sym[k] = 1;          // a function of u^2 + v^2
    double n = im.live_par[0] >= 0 ? prep_theta(p, io, im.live_par[0]) : im.live_fixed[0];
    double rd = im.live_par[1] >= 0 ? prep_theta(p, io, im.live_par[1]) : im.live_fixed[1];
    const bool valid = isfinite(n) && isfinite(rd) && n >= PSF_N_MIN && n <= PSF_N_MAX &&
                       rd >= PSF_RD_MIN && rd <= PSF_RD_MAX;
    if (!valid) {
        if (threadIdx.x == 0) {
            if (lm_trial) atomicOr(&p.lmf[im.sub].trial_bad, 1);
            else atomicOr(p.sticky, FLAG_DOMAIN);
        }
        n = 1.0;                                   // keeps the (unused) stamp finite
        rd = 1.0;
    }
    const double ird2 = 1.0 / (rd * rd);
    double sf = 0.0, sdn = 0.0, sdr = 0.0;
    for (int e = threadIdx.x; e < P2; e += blockDim.x) {
        const double u = (double)(e / P - c), v = (double)(e % P - c);
        const double r2 = u * u + v * v;
        const double x = 1.0 + r2 * ird2;
        const double f = exp(-n * log(x));
        sf += f;
        sdn += -log(x) * f;
        sdr += f * (-n) / x * (-2.0 * r2 * ird2 / rd);
    }
    for (int o = 32; o > 0; o >>= 1) {
        sf += __shfl_xor(sf, o, 64);
        sdn += __shfl_xor(sdn, o, 64);
        sdr += __shfl_xor(sdr, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6][0] = sf;
        red[threadIdx.x >> 6][1] = sdn;
        red[threadIdx.x >> 6][2] = sdr;
    }
    __syncthreads();
    const double S = ((red[0][0] + red[1][0]) + red[2][0]) + red[3][0];
    const double Sdn = ((red[0][1] + red[1][1]) + red[2][1]) + red[3][1];
    const double Sdr = ((red[0][2] + red[1][2]) + red[2][2]) + red[3][2];
    const double iS = 1.0 / S;
    float* K32 = p.psf_live + im.live_off;
    for (int e = threadIdx.x; e < P2; e += blockDim.x) {
        const double u = (double)(e / P - c), v = (double)(e % P - c);
        const double r2 = u * u + v * v;
        const double x = 1.0 + r2 * ird2;
        const double f = exp(-n * log(x));
        const double Kv = f * iS;
        const double dn = (-log(x) * f - Kv * Sdn) * iS;
        const double dr = (f * (-n) / x * (-2.0 * r2 * ird2 / rd) - Kv * Sdr) * iS;
        K64[e] = Kv;
        K32[e] = (float)Kv;
        if (io.flip) p.psf_flip[im.psf_off + P2 - 1 - e] = (float)Kv;
        K32[P2 + e] = (float)dn;
        K32[2 * P2 + e] = (float)dr;
    }
}

__global__ __launch_bounds__(256) void k_prep(PlanPtr pp, PrepIO io, PrepBlocks nb) {
    PlanRef p = *pp;
    int b = (int)blockIdx.x;
    if (b < nb.comps) {
        prep_comp(p, io, b * 256 + (int)threadIdx.x);
        return;
    }
    b -= nb.comps;
    if (b < nb.psf) {
        prep_psf(p, io, b);
        return;
    }
    b -= nb.psf;
    if (b < nb.begin) {
        if (io.adopt) {
            lm_adopt_sub(p, io.lm, b);
        } else {
            const int s = b * 256 + (int)threadIdx.x;
            if (s < p.n_sub) lm_begin_sub(p, io.lm, s);
        }
        return;
    }
    b -= nb.begin;
    const int k = b * 256 + (int)threadIdx.x;
    if (k < p.n_par) p.theta_trial[k] = prep_theta(p, io, k);
}

hipError_t launch_prep(const Plan& p, const PrepIO& io, hipStream_t st) {
    const int n = p.n_comps > p.n_images ? p.n_comps : p.n_images;
    PrepBlocks nb;
    nb.comps = (n + 255) / 256;
    nb.psf = p.n_images;
    nb.begin = !io.lm ? 0 : io.adopt ? p.n_sub : (p.n_sub + 255) / 256;
    nb.trial = io.step ? (p.n_par + 255) / 256 : 0;
    hipLaunchKernelGGL(k_prep, dim3(nb.comps + nb.psf + nb.begin + nb.trial), dim3(256), 0, st, p.dev, io, nb);
    return hipGetLastError();
}

// ------------------------------------------------------------------ samples
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float sersic_I(const CompConst& c, float dx, float dy) {
    const float xp = fmaf(dx, c.cs, dy * c.sn);
    const float yq = fmaf(dy, c.cs, -dx * c.sn) * c.iq;
    const float R2 = fmaxf(fmaf(xp, xp, yq * yq), 1e-12f);
    const double lt = fma((double)c.g, (double)fast_log2(R2), -c.h_d);
    const float t = fast_exp2((float)lt);
    return fast_exp2((float)fma(-c.B_d, (double)t, c.A_d));
}

// Adds wgt * dI/dtheta_k (k = x0, y0, q, PA, n, Re, log10 Ie) into acc.
// ... at a point given in the component's frame (xp along the major axis, yp across it)
__device__ __forceinline__ void sersic_dI_r(const CompConst& c, float xp, float yp, float wgt, float acc[7]) {
    const float yq = yp * c.iq;
    float R2 = fmaf(xp, xp, yq * yq);
    const bool floored = R2 < 1e-12f;
    R2 = floored ? 1e-12f : R2;
    const float lt = (float)fma((double)c.g, (double)fast_log2(R2), -c.h_d);
    const float t = fast_exp2(lt);
    const float I = fast_exp2((float)fma(-c.B_d, (double)t, c.A_d)) * wgt;
    const float inv_n = 2.f * c.g;
    // dI/dR divided by R (hardware reciprocals, 1 ulp: these derivative images feed the
    // FP32 Jacobian and adjoint, held to 3e-5 of each column's scale)
    const float bt = I * c.b * t * inv_n;
    const float G = floored ? 0.f : -bt * __builtin_amdgcn_rcpf(R2);
    const float dxp = G * xp;                 // dI/dx'
    const float dyp = G * yq * c.iq;          // dI/dy' = G y' / q^2
    acc[0] += -c.cs * dxp + c.sn * dyp;
    acc[1] += -c.sn * dxp - c.cs * dyp;
    acc[2] += -G * yq * yq * c.iq;            // dR/dq = -y'^2 / (q^3 R)
    acc[3] += G * xp * yp * (1.f - c.iq * c.iq);
    acc[4] += I * (c.bp * (1.f - t) + c.b * t * lt * LN2F * inv_n);
    acc[5] += bt * __builtin_amdgcn_rcpf(c.re);
    acc[6] += I * LN10F;
}

__device__ __forceinline__ void sersic_dI(const CompConst& c, float dx, float dy, float wgt,
                                          float acc[7]) {
    sersic_dI_r(c, fmaf(dx, c.cs, dy * c.sn), fmaf(dy, c.cs, -dx * c.sn), wgt, acc);
}

struct NodeSet {
    int s, rule, mode;
    float o[MAX_NODES_1D], w[MAX_NODES_1D];
};

// R < k Re at a pixel centre, as sqrt(xp^2 + (yp / q)^2) < k Re rounds it.  Outside a margin of
// 1e-12 about the isophote (thousands of roundings) the squares decide, without the division
// and the square root, which only pixels inside the margin pay for.
__device__ __forceinline__ bool within_kre(const CompConst& c, double ucx, double ucy) {
    const double dx = ucx - c.x0, dy = ucy - c.y0;
    const double xp = along64(c, dx, dy), yp = across64(c, dx, dy);
    const double ya = yp * c.iq_d;
    const double R2 = xp * xp + ya * ya, k2 = c.kre * c.kre;
    if (R2 < k2 * (1.0 - 1e-12)) return true;
    if (R2 > k2 * (1.0 + 1e-12)) return false;
    const double yq = yp / c.q_d;
    return sqrt(xp * xp + yq * yq) < c.kre;
}

// Pixel value (before the area factor) of a Sersic component.
__device__ __forceinline__ float sersic_pixel(PlanRef p, const CompConst& c, const DImage& im,
                                              double ucx, double ucy) {
    const float dxc = (float)(ucx - c.x0), dyc = (float)(ucy - c.y0);
    if (p.mode == APX_MODE_WITHIN_K_RE && !within_kre(c, ucx, ucy)) return sersic_I(c, dxc, dyc);
    const float a1 = (float)im.aff[1], a2 = (float)im.aff[2], a4 = (float)im.aff[4], a5 = (float)im.aff[5];
    float sum = 0.f;
    for (int ky = 0; ky < p.s; ++ky) {
        const float oy = p.node_o[ky], wy = p.node_w[ky];
        float row = 0.f;
        for (int kx = 0; kx < p.s; ++kx) {
            const float ox = p.node_o[kx];
            row = fmaf(p.node_w[kx], sersic_I(c, dxc + fmaf(a1, ox, a2 * oy), dyc + fmaf(a4, ox, a5 * oy)), row);
        }
        sum = fmaf(wy, row, sum);
    }
    return sum;
}

// Window-pixel index of (y, x) in the adaptive-integration arrays.
__device__ __forceinline__ long long adapt_index(const DComp& cp, int y, int x) {
    return cp.aoff + (long long)(y - cp.box[0]) * (cp.box[3] - cp.box[1]) + (x - cp.box[1]);
}

__device__ __forceinline__ void sersic_pixel_grad(PlanRef p, const CompConst& c, const DImage& im,
                                                  const DComp& cp, int y, int x, double ucx, double ucy,
                                                  float acc[7]) {
    for (int k = 0; k < 7; ++k) acc[k] = 0.f;
    const float dxc = (float)(ucx - c.x0), dyc = (float)(ucy - c.y0);
    if (p.mode == APX_MODE_WITHIN_K_RE && !within_kre(c, ucx, ucy)) {
        sersic_dI(c, dxc, dyc, 1.f, acc);
        return;
    }
    if (p.mode == APX_MODE_ADAPTIVE) {
        // the rule chosen at this theta: centre, 3 x 3 (the s x s nodes below), or refined
        const int code = p.acode[adapt_index(cp, y, x)];
        if (code == 0) {
            sersic_dI(c, dxc, dyc, 1.f, acc);
            return;
        }
        if (code < 0) {
            const long long r = -1LL - code;          // refine entry (always < n_apix)
            const float* dv = p.adval + 7LL * (r < p.n_apix ? r : 0);
            for (int k = 0; k < 7; ++k) acc[k] = r < p.n_apix ? dv[k] : __builtin_nanf("");
            return;
        }
    }
    // the nodes in the component's frame: (xp, yp) = (xp0 + ox ax + oy bx, yp0 + ox ay + oy by)
    // with (ax, ay), (bx, by) the pixel axes mapped and rotated once
    const float a1 = (float)im.aff[1], a2 = (float)im.aff[2], a4 = (float)im.aff[4], a5 = (float)im.aff[5];
    const float xp0 = fmaf(dxc, c.cs, dyc * c.sn), yp0 = fmaf(dyc, c.cs, -dxc * c.sn);
    const float ax = fmaf(a1, c.cs, a4 * c.sn), ay = fmaf(a4, c.cs, -a1 * c.sn);
    const float bx = fmaf(a2, c.cs, a5 * c.sn), by = fmaf(a5, c.cs, -a2 * c.sn);
    for (int ky = 0; ky < p.s; ++ky) {
        const float oy = p.node_o[ky];
        const float xr = fmaf(oy, bx, xp0), yr = fmaf(oy, by, yp0);
        for (int kx = 0; kx < p.s; ++kx) {
            const float ox = p.node_o[kx];
            sersic_dI_r(c, fmaf(ox, ax, xr), fmaf(ox, ay, yr), p.node_w[kx] * p.node_w[ky], acc);
        }
    }
}

__device__ __forceinline__ double point_weight(const CompConst& c, int y, int x) {
    const double wx = fmax(0.0, 1.0 - fabs((double)x - c.x0));
    const double wy = fmax(0.0, 1.0 - fabs((double)y - c.y0));
    return wx * wy;
}

// The same pixel integral in double precision throughout (FP64 log2/exp2), for the
// objective path: chi^2 differences of the LM gain ratio are resolved far below FP32
// rounding.
// tab: the 2^x / log2 table in LDS (PTAB_N doubles)
// The nodes of a pixel in the component's frame: the node at pixel offset (ox, oy) sits at
// (xp, yq) = (xp0 + ox ax + oy bx, yq0 + ox ay + oy by), with (xp0, yq0) the pixel centre's
// rotated and 1/q-scaled offset and (ax, ay), (bx, by) the images of the pixel axes (the
// affine map's columns rotated and scaled the same way, by k_prep): two FMAs per node instead
// of mapping and rotating every node.
//
// Away from the component's centre a node's R^2 = v0 (1 + d) is close to the pixel centre's
// v0, and t = (R / Re)^(1/n) follows from the centre's t0 by the binomial series of
// (1 + d)^g, g = 1/(2n), instead of a log2 and a 2^x of its own: 28 FP64 instructions per node
// instead of 49, and one log2 and one 2^x per pixel.  d = (linear + quadratic form of the
// offset) / v0 is formed without cancellation, so t carries no more rounding than before.
// DEG terms are taken while |d| <= bin_rho(DEG), where the rest is below 1.4e-16
// (|C(g, k)| < 0.016 at k = 8, < 0.0094 at k = 12 for g = 1/(2n), n in [0.36, 10]); the bound on
// |d| over the nodes must hold on every active lane of the wave, so the branch is uniform.
// Bound by FP64 issue; the full render of 768 cutouts (70 154 tiles of 8 x 32) goes from 821
// to 626 us, a 187 x 301 image with 4 x 4 Gauss-Legendre nodes from 49 to 32 us.
constexpr double bin_rho(int deg) { return deg == BIN_DEG ? 0.07 : 0.015; }
constexpr int BIN_DEG_FAR = 7;

template <int DEG, int S>
__device__ __forceinline__ double pixel64_series(PlanRef p, const CompConst& c, double iv, double gx, double gy,
                                                 double B0, double X0, const double* __restrict__ tab) {
    const double ux = gx * iv, uy = gy * iv, wxx = c.qxx * iv, wxy = c.qxy * iv, wyy = c.qyy * iv;
    const double nB = -64.0 * B0, X64 = 64.0 * X0;   // exponents in units of 1/64
    const double cl = vcopy64(c.bin[DEG - 1]), e4 = vcopy64(EXP2S_C4);
    const int s = S > 0 ? S : p.s;
    double sum = 0.0;
    auto node = [&](double ox, double base, double lin) {
        const double d = fma(ox, fma(ox, wxx, lin), base);
        double q = fma_vvs(cl, d, c.bin[DEG - 2]);
#pragma unroll
        for (int k = DEG - 3; k >= 0; --k) q = fma_vvs(q, d, c.bin[k]);
        return exp2_64th(fma(nB * d, q, X64), tab, e4);
    };
    auto line = [&](double oy, double wy) {
        const double base = oy * fma(oy, wyy, uy), lin = fma(oy, wxy, ux);
        double row = 0.0;
        if constexpr (S > 0) {
#pragma unroll
            for (int kx = 0; kx < S; ++kx) row = fma(p.node_wd[kx], node(p.node_od[kx], base, lin), row);
        } else {
            for (int kx = 0; kx < s; ++kx) row = fma(p.node_wd[kx], node(p.node_od[kx], base, lin), row);
        }
        sum = fma(wy, row, sum);
    };
    if constexpr (S > 0) {
#pragma unroll
        for (int ky = 0; ky < S; ++ky) line(p.node_od[ky], p.node_wd[ky]);
    } else {
        for (int ky = 0; ky < s; ++ky) line(p.node_od[ky], p.node_wd[ky]);
    }
    return sum;
}

template <int S, bool FIT>
__device__ __forceinline__ double pixel64_nodes(PlanRef p, const CompConst& c, double xp0, double yq0,
                                                const double* __restrict__ tab) {
    const Poly64Regs rg = poly64_regs(c);
    const double v0 = xp0 * xp0 + yq0 * yq0;
    const double gx = 2.0 * (xp0 * c.ax + yq0 * c.ay), gy = 2.0 * (xp0 * c.bx + yq0 * c.by);
    const double dv = fma(fabs(gx) + fabs(gy), p.node_max, c.qmax);     // bounds v0 |d|
    // (v0 far enough above the floor of R^2 that no node reaches it; false for a NaN)
    if (!FIT && __all(dv <= bin_rho(BIN_DEG) * v0 && v0 >= 4e-12)) {
        const double B0 = c.B_d * exp2_t<false>(fma(c.g_d, log2_t(v0, tab, rg), -rg.h), tab, rg);
        const double X0 = rg.A - B0;
        // exponents that need no clamp: |X0 - B0 ((1 + d)^g - 1)| < 1000
        if (__all(B0 < 900.0 && fabs(X0) < 900.0)) {
            double iv = __builtin_amdgcn_rcp(v0);
            iv = fma(iv, fma(-v0, iv, 1.0), iv);
            iv = fma(iv, fma(-v0, iv, 1.0), iv);
            if (__all(dv <= bin_rho(BIN_DEG_FAR) * v0))
                return pixel64_series<BIN_DEG_FAR, S>(p, c, iv, gx, gy, B0, X0, tab);
            return pixel64_series<BIN_DEG, S>(p, c, iv, gx, gy, B0, X0, tab);
        }
    }
    double sum = 0.0;
    auto line = [&](double oy, double wy) {
        const double xr = fma(oy, c.bx, xp0), yr = fma(oy, c.by, yq0);
        double row = 0.0;
        if constexpr (S > 0) {
#pragma unroll
            for (int kx = 0; kx < S; ++kx)
                row += p.node_wd[kx] * sersic_I64_r(c, fma(p.node_od[kx], c.ax, xr), fma(p.node_od[kx], c.ay, yr), tab, rg);
        } else {
            for (int kx = 0; kx < p.s; ++kx)
                row += p.node_wd[kx] * sersic_I64_r(c, fma(p.node_od[kx], c.ax, xr), fma(p.node_od[kx], c.ay, yr), tab, rg);
        }
        sum += wy * row;
    };
    if constexpr (S > 0) {
#pragma unroll
        for (int ky = 0; ky < S; ++ky) line(p.node_od[ky], p.node_wd[ky]);
    } else {
        for (int ky = 0; ky < p.s; ++ky) line(p.node_od[ky], p.node_wd[ky]);
    }
    return sum;
}

template <bool FIT>
__device__ __forceinline__ double sersic_pixel64(PlanRef p, const CompConst& c, double ucx, double ucy,
                                                 const double* __restrict__ tab) {
    const double dxc = ucx - c.x0, dyc = ucy - c.y0;
    if (p.mode == APX_MODE_WITHIN_K_RE && !within_kre(c, ucx, ucy)) return sersic_I64_t(c, dxc, dyc, tab);
    const double xp0 = along64(c, dxc, dyc), yq0 = across64(c, dxc, dyc) * c.iq_d;
    // the usual rules unrolled (a loop waits for its node's scalar loads at every node)
    switch (p.s) {
        case 2: return pixel64_nodes<2, FIT>(p, c, xp0, yq0, tab);
        case 3: return pixel64_nodes<3, FIT>(p, c, xp0, yq0, tab);
        case 4: return pixel64_nodes<4, FIT>(p, c, xp0, yq0, tab);
        default: return pixel64_nodes<0, FIT>(p, c, xp0, yq0, tab);
    }
}

// Stage the 2^x / log2 table into LDS (the caller synchronises before use).
__device__ __forceinline__ void stage_ptab(PlanRef p, double* sh) {
    for (int k = (int)threadIdx.x; k < PTAB_N; k += (int)blockDim.x) sh[k] = p.ptab[k];
}

// ------------------------------------------------------------- re-centred tiles
// A re-centred Sersic (§2.1.3) enters the pre-convolution grid as T * S': S' sampled with
// the centre at the nearest pixel centre, T the separable interpolation taps (the shift
// commutes with the PSF convolution).  A workgroup owning an RT_Y x RT_X tile with origin
// (y0, x0) samples S' once over the tile grown by a on every side into LDS (zero outside
// the sampled window sbox), then every pixel sums its (2a+1)^2 taps from LDS.
constexpr int SH_H = RT_Y + 2 * APX_SHIFT_MAX_A, SH_W = RT_X + 2 * APX_SHIFT_MAX_A;

// Stage NPL planes of f(ry, rx, out[NPL]) over the grown tile, sh[q][hy * (RT_X + 2a) + hx],
// and the component's taps into tw (wx, wy, dwx, dwy; SHIFT_NT each).  The caller
// synchronises before reading them.
template <int NPL, typename T, typename F>
__device__ __forceinline__ void stage_halo(PlanRef p, int ci, const DComp& cp, int y0, int x0,
                                           T (*sh)[SH_H * SH_W], T* tw, F&& f) {
    const int a = p.shift_a, HW = RT_X + 2 * a, n = (RT_Y + 2 * a) * HW;
    if (threadIdx.x < STAP_STRIDE) tw[threadIdx.x] = (T)p.stap[(long long)ci * STAP_STRIDE + threadIdx.x];
    for (int e = (int)threadIdx.x; e < n; e += 256) {
        const int hy = e / HW, hx = e - hy * HW;
        const int ry = y0 - a + hy, rx = x0 - a + hx;
        T v[NPL];
        for (int q = 0; q < NPL; ++q) v[q] = (T)0;
        if (ry >= cp.sbox[0] && ry < cp.sbox[2] && rx >= cp.sbox[1] && rx < cp.sbox[3]) f(ry, rx, v);
        for (int q = 0; q < NPL; ++q) sh[q][e] = v[q];
    }
}

// sum_t wy[ty] wx[tx] plane(ly - ty, lx - tx) for the pixel (ly, lx) of the tile (taps in
// LDS, the same for every thread); unrolled per half-width A.
template <int A, typename T>
__device__ __forceinline__ T tap_sum_a(const T* plane, int ly, int lx, const T* wy, const T* wx) {
    constexpr int HW = RT_X + 2 * A;
    const T* base = plane + (ly + 2 * A) * HW + lx + 2 * A;
    T out = (T)0;
#pragma unroll
    for (int jy = 0; jy <= 2 * A; ++jy) {
        const T* row = base - jy * HW;
        T acc = (T)0;
#pragma unroll
        for (int jx = 0; jx <= 2 * A; ++jx) acc = fma(wx[jx], row[-jx], acc);
        out = fma(wy[jy], acc, out);
    }
    return out;
}

template <typename T>
__device__ __forceinline__ T tap_sum(const T* plane, int a, int ly, int lx, const T* wy, const T* wx) {
    switch (a) {
        case 1: return tap_sum_a<1>(plane, ly, lx, wy, wx);
        case 2: return tap_sum_a<2>(plane, ly, lx, wy, wx);
        case 3: return tap_sum_a<3>(plane, ly, lx, wy, wx);
        case 4: return tap_sum_a<4>(plane, ly, lx, wy, wx);
        default: return tap_sum_a<5>(plane, ly, lx, wy, wx);
    }
}

// The 7 pre-convolution derivative values (area included: it is in the staged planes) of
// a re-centred Sersic at pixel (ly, lx) of a tile whose origin is (y0, x0):
// d/d(q, PA, n, Re, log Ie) are T * dS'/dtheta; x0 and y0 move only delta, so
// d/d x0 = inv1 (dT/d delta_x * S') + inv4 (dT/d delta_y * S') (inv2, inv5 for y0), with
// S' = (d/d log Ie plane) / ln 10.  Every thread of the block calls it.
__device__ void shifted_derivs(PlanRef p, int ci, const CompConst& c, const DComp& cp, const DImage& im,
                               int y0, int x0, int ly, int lx, bool want, float (*sh)[SH_H * SH_W],
                               float* tw, float out[7]) {
    stage_halo<5, float>(p, ci, cp, y0, x0, sh, tw, [&](int ry, int rx, float* v) {
        const double ucx = im.aff[0] + im.aff[1] * rx + im.aff[2] * ry;
        const double ucy = im.aff[3] + im.aff[4] * rx + im.aff[5] * ry;
        float acc[7];
        sersic_pixel_grad(p, c, im, cp, ry, rx, ucx, ucy, acc);
        const float area = (float)im.area;
        for (int q = 0; q < 5; ++q) v[q] = acc[q + 2] * area;
    });
    __syncthreads();
    for (int q = 0; q < 7; ++q) out[q] = 0.f;
    if (want) {
        const float *wx = tw, *wy = tw + SHIFT_NT, *dwx = tw + 2 * SHIFT_NT, *dwy = tw + 3 * SHIFT_NT;
        const int a = p.shift_a;
        for (int q = 0; q < 5; ++q) out[q + 2] = tap_sum(sh[q], a, ly, lx, wy, wx);
        const float inv_ln10 = 1.f / LN10F;
        const float mx = tap_sum(sh[4], a, ly, lx, wy, dwx) * inv_ln10;
        const float my = tap_sum(sh[4], a, ly, lx, dwy, wx) * inv_ln10;
        out[0] = (float)im.inv[1] * mx + (float)im.inv[4] * my;
        out[1] = (float)im.inv[2] * mx + (float)im.inv[5] * my;
    }
    __syncthreads();
}

// Pixel value T * S' (area included) of a re-centred Sersic at pixel (ly, lx) of the render
// tile with origin (y0, x0); 0 where !want.  Every thread of the block calls it.
template <typename T, bool FIT>
__device__ T shifted_pixel(PlanRef p, int ci, const CompConst& c, const DComp& cp, const DImage& im, int y0,
                           int x0, int ly, int lx, bool want, T (*sh)[SH_H * SH_W], T* tw,
                           const double* __restrict__ tab = nullptr) {
    stage_halo<1, T>(p, ci, cp, y0, x0, sh, tw, [&](int ry, int rx, T* v) {
        const double rcx = im.aff[0] + im.aff[1] * rx + im.aff[2] * ry;
        const double rcy = im.aff[3] + im.aff[4] * rx + im.aff[5] * ry;
        if constexpr (sizeof(T) == 8) v[0] = sersic_pixel64<FIT>(p, c, rcx, rcy, tab) * im.area;
        else v[0] = (float)((double)sersic_pixel(p, c, im, rcx, rcy) * im.area);
    });
    __syncthreads();
    const T out = want ? tap_sum(sh[0], p.shift_a, ly, lx, tw + SHIFT_NT, tw) : (T)0;
    __syncthreads();
    return out;
}

// ----------------------------------------------------------------------- render
// S (extended grid) = sum of all components whose window holds the pixel.
// SHIFT: the problem re-centres its Sersics (a separate instantiation keeps the plain
// kernels' register and LDS budgets)
template <bool SHIFT>
__global__ __launch_bounds__(256) void k_render(PlanPtr pp, int skip_mode, const apx_lm_state* lm) {
    PlanRef p = *pp;
    __shared__ float sh[1][SHIFT ? SH_H * SH_W : 1];
    __shared__ float tw[SHIFT ? STAP_STRIDE : 1];
    const RTile t = p.rtiles[blockIdx.x];
    const DImage& im = p.images[t.a];
    if (sub_skipped(p, im.sub, skip_mode, lm)) return;
    const int ly = (int)threadIdx.x / RT_X, lx = (int)threadIdx.x % RT_X;
    const int y = t.y0 + ly, x = t.x0 + lx;
    const bool inside = y < im.H + im.c && x < im.W + im.c;
    const double ucx = im.aff[0] + im.aff[1] * x + im.aff[2] * y;
    const double ucy = im.aff[3] + im.aff[4] * x + im.aff[5] * y;
    double sum = 0.0;
    const int kb = p.rtile_off[blockIdx.x], ke = p.rtile_off[blockIdx.x + 1];
    for (int k = kb; k < ke; ++k) {
        const int ci = p.rtile_comps[k];
        const DComp& cp = p.comps[ci];
        const bool inbox = inside && y >= cp.box[0] && y < cp.box[2] && x >= cp.box[1] && x < cp.box[3];
        const CompConst& c = p.cc[ci];
        if (!c.valid) {
            if (inbox) sum += __builtin_nan("");
            continue;
        }
        if (SHIFT && cp.type == APX_SERSIC) {      // block-uniform
            if constexpr (SHIFT) sum += (double)shifted_pixel<float, false>(p, ci, c, cp, im, t.y0, t.x0, ly, lx, inbox, sh, tw);
            continue;
        }
        if (!inbox) continue;
        if (cp.type == APX_SERSIC)
            sum += (p.mode == APX_MODE_ADAPTIVE ? p.aval[adapt_index(cp, y, x)]
                                                : (double)sersic_pixel(p, c, im, ucx, ucy)) * im.area;
        else sum += (double)c.F * point_weight(c, y, x);
    }
    if (inside) p.S[im.ext_off + (long long)(y + im.c) * im.EW + (x + im.c)] = (float)sum;
}

hipError_t launch_render_mode(const Plan& p, int skip_mode, const apx_lm_state* lm, hipStream_t st) {
    if (p.n_rtiles == 0) return hipSuccess;
    if (p.shift != APX_SHIFT_NONE)
        hipLaunchKernelGGL(k_render<true>, dim3(p.n_rtiles), dim3(256), 0, st, p.dev, skip_mode, lm);
    else
        hipLaunchKernelGGL(k_render<false>, dim3(p.n_rtiles), dim3(256), 0, st, p.dev, skip_mode, lm);
    return hipGetLastError();
}

// ------------------------------------------------------------- FP64 render
// S64 (extended grid, FP64): the objective path's render.  FIT (the evaluations of an LM fit):
// every node by its own log2 and 2^x, without the series of pixel64_series.  Both carry the
// same rounding error, but they do not round alike, and a fit follows the last bits of its
// residuals: a theta that moves by 1e-14 turns the rounding of a few nodes of the FP32
// derivative images, which changes the rounding of their whole FFT tiles (1e-8 of J^T W r), and
// two iterations later the largest parameter of 768 cutouts by 1e-5.  So a fit keeps the one
// arithmetic it has always had, and its result.  (A full render of 768 cutouts: 821 us, with the
// series 626.)
template <bool SHIFT, bool FIT>
__global__ __launch_bounds__(256, SHIFT || FIT ? 4 : 6) void k_render64(PlanPtr pp, int skip_mode, const apx_lm_state* lm) {
    PlanRef p = *pp;
    __shared__ double sh[1][SHIFT ? SH_H * SH_W : 1];
    __shared__ double tw[SHIFT ? STAP_STRIDE : 1];
    __shared__ double ptab[PTAB_N];
    const RTile t = p.rtiles[blockIdx.x];
    const DImage& im = p.images[t.a];
    if (sub_skipped(p, im.sub, skip_mode, lm)) return;
    stage_ptab(p, ptab);
    __syncthreads();
    const int ly = (int)threadIdx.x / RT_X, lx = (int)threadIdx.x % RT_X;
    const int y = t.y0 + ly, x = t.x0 + lx;
    const bool inside = y < im.H + im.c && x < im.W + im.c;
    const double ucx = im.aff[0] + im.aff[1] * x + im.aff[2] * y;
    const double ucy = im.aff[3] + im.aff[4] * x + im.aff[5] * y;
    double sum = 0.0;
    const int kb = p.rtile_off[blockIdx.x], ke = p.rtile_off[blockIdx.x + 1];
    for (int k = kb; k < ke; ++k) {
        const int ci = p.rtile_comps[k];
        const DComp& cp = p.comps[ci];
        const bool inbox = inside && y >= cp.box[0] && y < cp.box[2] && x >= cp.box[1] && x < cp.box[3];
        const CompConst& c = p.cc[ci];
        if (!c.valid) {
            if (inbox) sum += __builtin_nan("");
            continue;
        }
        if (SHIFT && cp.type == APX_SERSIC) {      // block-uniform
            if constexpr (SHIFT) sum += shifted_pixel<double, FIT>(p, ci, c, cp, im, t.y0, t.x0, ly, lx, inbox, sh, tw, ptab);
            continue;
        }
        if (!inbox) continue;
        if (cp.type == APX_SERSIC)
            sum += (p.mode == APX_MODE_ADAPTIVE ? p.aval[adapt_index(cp, y, x)]
                                                : sersic_pixel64<FIT>(p, c, ucx, ucy, ptab)) * im.area;
        else sum += (double)c.F64 * point_weight(c, y, x);
    }
    if (inside) p.S64[im.ext_off + (long long)(y + im.c) * im.EW + (x + im.c)] = sum;
}

hipError_t launch_render64(const Plan& p, int fit, int skip_mode, const apx_lm_state* lm, hipStream_t st) {
    if (p.n_rtiles == 0) return hipSuccess;
    auto* k = p.shift != APX_SHIFT_NONE ? (fit ? k_render64<true, true> : k_render64<true, false>)
                                        : (fit ? k_render64<false, true> : k_render64<false, false>);
    hipLaunchKernelGGL(k, dim3(p.n_rtiles), dim3(256), 0, st, p.dev, skip_mode, lm);
    return hipGetLastError();
}

// ------------------------------------------------------------ derivative images
// D[col] over the group's input box: the pixel-integrated derivative of each free
// parameter of each component of the group (pre-convolution).
template <bool SHIFT>
__global__ __launch_bounds__(256) void k_deriv(PlanPtr pp, const apx_lm_state* lm) {
    PlanRef p = *pp;
    __shared__ float sh[5][SHIFT ? SH_H * SH_W : 1];
    __shared__ float tw[SHIFT ? STAP_STRIDE : 1];
    const RTile t = p.gtiles[blockIdx.x];
    const DGroup& gr = p.groups[t.a];
    if (gr.comp_begin + (int)blockIdx.y >= gr.comp_end) return;
    if (lm && lm[gr.sub].need_jac == 0) return;
    const DImage& im = p.images[gr.image];
    const int ty = (int)threadIdx.x / RT_X, tx = (int)threadIdx.x % RT_X;
    const int ly = t.y0 + ty, lx = t.x0 + tx;
    const bool inside = ly < gr.ih && lx < gr.iw;
    const int y = gr.iy0 + ly, x = gr.ix0 + lx;
    const double ucx = im.aff[0] + im.aff[1] * x + im.aff[2] * y;
    const double ucy = im.aff[3] + im.aff[4] * x + im.aff[5] * y;
    const long long plane = (long long)gr.ih * gr.iw;
    float* Dg = p.D + gr.d_off + (long long)ly * gr.iw + lx;
    for (int k = gr.comp_begin + (int)blockIdx.y; k < gr.comp_end; k += (int)gridDim.y) {
        const int ci = p.group_comps[k];
        const DComp& cp = p.comps[ci];
        const CompConst& c = p.cc[ci];
        if (SHIFT && cp.type == APX_SERSIC) {      // block-uniform
            float acc[7] = {};
            if constexpr (SHIFT)
                shifted_derivs(p, ci, c, cp, im, gr.iy0 + t.y0, gr.ix0 + t.x0, ty, tx, inside, sh, tw, acc);
            if (inside)
                for (int q = 0; q < 7; ++q)
                    if (cp.col[q] >= 0) Dg[cp.col[q] * plane] = acc[q];
            continue;
        }
        if (!inside) continue;
        if (cp.type == APX_SERSIC) {
            float acc[7];
            sersic_pixel_grad(p, c, im, cp, y, x, ucx, ucy, acc);
            const float area = (float)im.area;
            for (int q = 0; q < 7; ++q)
                if (cp.col[q] >= 0) Dg[cp.col[q] * plane] = acc[q] * area;
        } else {
            if (cp.col[2] >= 0) Dg[cp.col[2] * plane] = (float)((double)c.F * point_weight(c, y, x) * 2.302585092994046);
        }
    }
}

hipError_t launch_deriv(const Plan& p, const apx_lm_state* lm, hipStream_t st) {
    if (p.n_gtiles == 0) return hipSuccess;
    if (p.shift != APX_SHIFT_NONE)
        hipLaunchKernelGGL(k_deriv<true>, dim3(p.n_gtiles, p.g_split), dim3(256), 0, st, p.dev, lm);
    else
        hipLaunchKernelGGL(k_deriv<false>, dim3(p.n_gtiles, p.g_split), dim3(256), 0, st, p.dev, lm);
    return hipGetLastError();
}

// ------------------------------------------------------------- adjoint gradient
__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The sums of v[0..6] over the wave, v[q]'s in lanes 8 q .. 8 q + 7: lanes that differ in one
// bit of the lane halve the values they hold between them, then each sum finishes in its eight
// lanes.  10 exchanges of a double; a butterfly for each value takes 42.
__device__ __forceinline__ double wave_sum7(const double (&v)[7], int lane) {
    double a[4], b[2];
    const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double hi = k + 4 < 7 ? v[k + 4 < 7 ? k + 4 : 0] : 0.0;
        a[k] = (h5 ? hi : v[k]) + __shfl_xor(h5 ? v[k] : hi, 32, 64);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) b[k] = (h4 ? a[k + 2] : a[k]) + __shfl_xor(h4 ? a[k] : a[k + 2], 16, 64);
    double s = (h3 ? b[1] : b[0]) + __shfl_xor(h3 ? b[0] : b[1], 8, 64);
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    return s;
}

// grad_part[col][tile] = sum over the tile of Abar * dS/dtheta_col (recomputed).
template <bool SHIFT>
__global__ __launch_bounds__(256) void k_grad_tiles(PlanPtr pp) {
    PlanRef p = *pp;
    __shared__ double red[2][4][8];                // by turns: one barrier per component
    __shared__ float sh[5][SHIFT ? SH_H * SH_W : 1];
    __shared__ float tw[SHIFT ? STAP_STRIDE : 1];
    const RTile t = p.gtiles[blockIdx.x];
    const DGroup& gr = p.groups[t.a];
    if (gr.comp_begin + (int)blockIdx.y >= gr.comp_end) return;
    const DImage& im = p.images[gr.image];
    const int tile_local = blockIdx.x - gr.tile_begin;
    const int ly = t.y0 + (int)threadIdx.x / RT_X;
    const int lx = t.x0 + (int)threadIdx.x % RT_X;
    const bool inside = ly < gr.ih && lx < gr.iw;
    const int y = gr.iy0 + ly, x = gr.ix0 + lx;
    const double ucx = im.aff[0] + im.aff[1] * x + im.aff[2] * y;
    const double ucy = im.aff[3] + im.aff[4] * x + im.aff[5] * y;
    float abar = 0.f;
    if (inside) abar = p.Abar[im.ext_off + (long long)(y + im.c) * im.EW + (x + im.c)];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int turn = 0;
    for (int k = gr.comp_begin + (int)blockIdx.y; k < gr.comp_end; k += (int)gridDim.y) {
        const int ci = p.group_comps[k];
        const DComp& cp = p.comps[ci];
        const CompConst& c = p.cc[ci];
        double(&rd)[4][8] = red[turn];
        turn ^= 1;
        if (cp.type == APX_SERSIC) {               // block-uniform
            double v[7];
            float acc[7] = {};
            if constexpr (SHIFT) {
                shifted_derivs(p, ci, c, cp, im, gr.iy0 + t.y0, gr.ix0 + t.x0, ly - t.y0, lx - t.x0, inside, sh, tw,
                               acc);
                for (int q = 0; q < 7; ++q) v[q] = (double)acc[q] * (double)abar;
            } else {
                if (inside) sersic_pixel_grad(p, c, im, cp, y, x, ucx, ucy, acc);
                for (int q = 0; q < 7; ++q) v[q] = (double)acc[q] * im.area * (double)abar;
            }
            const double s = wave_sum7(v, lane);
            if ((lane & 7) == 0) rd[wv][lane >> 3] = s;
        } else if (cp.col[2] >= 0) {
            double v = 0.0;
            if (inside) v = (double)c.F * point_weight(c, y, x) * 2.302585092994046 * (double)abar;
            v = wave_sum(v);
            if (lane == 0) rd[wv][2] = v;
        }
        __syncthreads();
        if (threadIdx.x < 7 && cp.col[threadIdx.x] >= 0) {
            const int q = threadIdx.x;
            const double s = ((rd[0][q] + rd[1][q]) + rd[2][q]) + rd[3][q];
            p.grad_part[gr.gp_off + (long long)cp.col[q] * gr.ntiles + tile_local] = s;
        }
    }
}

hipError_t launch_grad_tiles(const Plan& p, hipStream_t st) {
    if (p.n_gtiles == 0) return hipSuccess;
    if (p.shift != APX_SHIFT_NONE)
        hipLaunchKernelGGL(k_grad_tiles<true>, dim3(p.n_gtiles, p.g_split), dim3(256), 0, st, p.dev);
    else
        hipLaunchKernelGGL(k_grad_tiles<false>, dim3(p.n_gtiles, p.g_split), dim3(256), 0, st, p.dev);
    return hipGetLastError();
}

// -------------------------------------------------------------- seed sums (VJP sky column)
// Block c of image k sums pixels c*256 + t + SEED_BLOCKS*256*m in FP64 (fixed order per
// thread, then waves in order); one wave per image folds the SEED_BLOCKS partials.
constexpr int SEED_BLOCKS = 64;
__global__ __launch_bounds__(256) void k_seed_part(PlanPtr pp, const float* __restrict__ seed, double* part) {
    PlanRef p = *pp;
    __shared__ double red[4];
    const int k = blockIdx.y, c = blockIdx.x;
    const DImage& im = p.images[k];
    const long long npx = (long long)im.Hc * im.Wc;
    double acc = 0.0;
    for (long long e = (long long)c * 256 + threadIdx.x; e < npx; e += (long long)SEED_BLOCKS * 256)
        acc += (double)seed[im.pix_off + e];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[k * SEED_BLOCKS + c] = ((red[0] + red[1]) + red[2]) + red[3];
}

__global__ void k_seed_fold(PlanPtr pp, const double* __restrict__ part) {
    PlanRef p = *pp;
    const int k = blockIdx.x;
    double v = part[k * SEED_BLOCKS + threadIdx.x];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (threadIdx.x == 0) p.img_sum[3 * k + 1] = -0.5 * v;
}

hipError_t launch_seed_sums(const Plan& p, const float* seed, double* part, hipStream_t st) {
    static_assert(SEED_BLOCKS == 64, "one lane per partial in the fold");
    if (p.n_images == 0) return hipSuccess;
    hipLaunchKernelGGL(k_seed_part, dim3(SEED_BLOCKS, p.n_images), dim3(256), 0, st, p.dev, seed, part);
    hipLaunchKernelGGL(k_seed_fold, dim3(p.n_images), dim3(64), 0, st, p.dev, part);
    return hipGetLastError();
}

}  // namespace apx
