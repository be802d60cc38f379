// Direct-mode PSF convolution (§2.1.3) for gfx950.
//
// out(y, x) = sum_{U,V} K[U][V] * in(y - U + c, x - V + c), in = 0 outside its rectangle.
//
// One workgroup owns a TH x TW output tile (TH * TW / R threads).  The input tile with its
// (P-1) halo is staged once into LDS; each lane then produces R consecutive outputs
// of one row: per PSF row it loads an R + P - 1 register window from LDS (ds_read_b128)
// and runs P x R FMAs whose PSF operand is wave-uniform (scalar loads, then copied to
// a VGPR), so the VALU does useful FMAs at ~R*P per (R+P-1)/4 LDS instructions.  Each PSF row is summed
// into a fresh partial before being added to the accumulator (error ~2P ulp, not P^2).
// R = CV_R = 8 where there are tiles enough to fill the chip; launches of few tiles take
// R = CV_R_FINE = 2 on 16 x 32 tiles (four times the lanes per output: one 128 x 128 image at
// P = 25 takes 11.8 us instead of 18 in FP32 and in FP64, where a full chip runs the R = 2
// kernel at 57 instead of 80 TFLOP/s).  The arithmetic of an output does not depend on R.
//
// On an image whose PSF has a higher resolution than its pixels the grid is of sub-pixels,
// and the model and Jacobian epilogues first sum each pixel's sub-pixel outputs.
//
// Epilogues (template KIND):
//   CONV_FWD  model + sky, optional model store, FP32 residual store, FP64 partials of
//             sum w r^2, sum w r, sum w (chi^2 of Eq. chi2, sky gradient, sky-sky entry);
//   CONV_JCOL Jacobian column store, FP64 partials of sum w r J, sum w J (only for jobs
//             without gram_part: the 4 x 4-block Gram kernel forms them for the others);
//   CONV_ADJ  input is -2 w r staged from the residual (the adjoint seed of chi^2), or a
//             given seed (vector-Jacobian product of the render), PSF flipped,
//             output is dchi2/dS on the extended grid.
#pragma once
#include <type_traits>

#include "apx_internal.h"

namespace apx {

// Sum of each run of UU consecutive entries into the first R / UU entries.
template <int UU, typename T, int R>
__device__ __forceinline__ void bin_lane(T (&acc)[R]) {
#pragma unroll
    for (int q = 0; q < R / UU; ++q) {
        T v = acc[q * UU];
#pragma unroll
        for (int i = 1; i < UU; ++i) v += acc[q * UU + i];
        acc[q] = v;
    }
}

__device__ __forceinline__ double conv_wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sub-pixel grids (up = U > 1, a power of two <= CV_R): sum each pixel's U x U outputs, U
// consecutive ones in a lane, then across the lanes of rows ty ^ 1 .. ty ^ (U - 1) (one wave
// holds 64 / LPR >= 8 rows; tiles and output boxes are whole pixels).  Lane rows with
// ty % U == 0 then hold R / U pixel values each.  Launches with R < CV_R hold no such image.
template <int LPR, typename T, int R>
__device__ __forceinline__ void bin_pixels(T (&acc)[R], int up) {
    if constexpr (R == CV_R) {
        if (up == 1) return;
        if (up == 2) bin_lane<2>(acc);
        else if (up == 4) bin_lane<4>(acc);
        else bin_lane<8>(acc);
        for (int k = 1; k < up; k <<= 1)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] += __shfl_xor(acc[r], k * LPR, 64);
    }
}

// Epilogue of the model convolution: model + sky, optional model store, FP32 residual store,
// FP64 partials of sum w r^2, sum w r, sum w per item.
template <typename T, int R, int NW>
__device__ __forceinline__ void fwd_epilogue(PlanRef p, const ConvJob& jb, const DImage& im, const ConvIO& io,
                                             int item_idx, const T (&acc)[R], int y, int xb, bool yok,
                                             double (*red)[3]) {
    const int up = im.up, nq = R / up;               // values per lane, render-grid step between them
    const int xend = jb.out_x0 + jb.out_w;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const T sky = (T)p.sky_val[jb.image];
    double c2 = 0.0, swr = 0.0, sw = 0.0;
    if (yok) {
        const long long rowpix = im.pix_off + (long long)(y / up) * im.Wc;
        // the row's weights and data first: their loads overlap instead of following
        // one another
        float wv[R], dv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int x = xb + r * up;
            wv[r] = dv[r] = 0.f;
            if (io.data && r < nq && x < xend) {
                wv[r] = io.weight[rowpix + x / up];
                dv[r] = io.data[rowpix + x / up];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int x = xb + r * up;
            if (r < nq && x < xend) {
                const T m = acc[r] + sky;
                const long long pix = rowpix + x / up;
                if (io.out) io.out[pix] = (float)m;
                if (io.data) {
                    const double w = (double)wv[r];
                    const double rr = (double)dv[r] - (double)m;
                    c2 += w * rr * rr;
                    swr += w * rr;
                    sw += w;
                    p.rbuf[pix] = (float)rr;
                }
            }
        }
    }
    if (io.data) {
        c2 = conv_wave_sum(c2);
        swr = conv_wave_sum(swr);
        sw = conv_wave_sum(sw);
        if (lane == 0) { red[wv][0] = c2; red[wv][1] = swr; red[wv][2] = sw; }
        __syncthreads();
        if (threadIdx.x < 3) {
            const int q = threadIdx.x;
            double sum = red[0][q];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += red[w][q];
            io.part[(long long)item_idx * 3 + q] = sum;
        }
    }
}

// Whether the sub-problem of an item skips this phase.
__device__ __forceinline__ bool conv_skipped(PlanRef p, const ConvIO& io, int sub) {
    if (io.skip_mode == 1) return p.lmf[sub].chol_done == 0 || p.lmf[sub].trial_bad != 0;
    if (io.skip_mode == 2) return io.lm[sub].need_jac == 0;
    return false;
}

// The stamp into LDS (rows KP long), for the fine tiles: a launch of few tiles has one wave or
// two per SIMD, too few to hide that each row's scalar loads of a stamp that another kernel has
// just written go out to the last-level cache; one round of vector loads beside the input's
// takes their place (a 128 x 128 gradient at P = 25: 17 -> 11 us per FP32 launch, 13.2 -> 12.6 in
// FP64, where LDS reads bound the rest).
template <int P, int KP, int NT, typename T>
__device__ inline void stage_stamp(T* __restrict__ kt, const T* __restrict__ K) {
    constexpr int NE = (P * P + NT - 1) / NT;
    T v[NE];
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const int e = (int)threadIdx.x + NT * q;
        v[q] = e < P * P ? K[e] : T(0);
    }
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const int e = (int)threadIdx.x + NT * q;
        if (e < P * P) kt[(e / P) * KP + e % P] = v[q];
    }
}

// The FP32 kinds.
template <int P, int KIND, int TH, int TW, int R>
__global__ __launch_bounds__(TH * TW / R) void k_conv(PlanPtr pp, const ConvJob* __restrict__ jobs,
                                                      const ConvItem* __restrict__ items, int item_begin,
                                                      ConvIO io) {
    PlanRef p = *pp;
    using T = float;
    constexpr int c = (P - 1) / 2;
    constexpr int NT = TH * TW / R;                 // threads
    constexpr int LPR = TW / R;                     // lanes per output row
    constexpr int NW = NT / 64;                     // waves
    static_assert(NW >= 1 && NT % 64 == 0, "whole waves");
    constexpr int LH = TH + P - 1;
    constexpr int LW0 = TW + P - 1;
    constexpr int LW = (LW0 + 3) & ~3;
    __shared__ __attribute__((aligned(16))) T tile[LH * LW];
    __shared__ double red[NW][3];
    constexpr bool KLDS = R != CV_R;
    constexpr int KP = (P + 3) & ~3;
    __shared__ __attribute__((aligned(16))) T kt[KLDS ? P * KP : 1];

    const int item_idx = item_begin + xcd_chunk_item((int)blockIdx.x, (int)gridDim.x);
    const ConvItem it = items[item_idx];
    const ConvJob jb = jobs[it.job];
    const DImage& im = p.images[jb.image];
    if (conv_skipped(p, io, im.sub)) return;
    const int oy0 = jb.out_y0 + it.ty * TH;
    const int ox0 = jb.out_x0 + it.tx * TW;
    const int iy_base = oy0 - c, ix_base = ox0 - c;
    // the stamp: the flipped stamp for the adjoint; on a live-PSF image the rendered stamp, or
    // for its PSF columns a derivative stamp
    const float* __restrict__ K;
    if constexpr (KIND == CONV_ADJ) K = p.psf_flip + im.psf_off;
    else K = im.live ? p.psf_live + im.live_off + (long long)jb.kslot[it.ch < 1 ? 0 : 1] * P * P
                     : p.psf + im.psf_off;
    if constexpr (KLDS) stage_stamp<P, KP, NT>(kt, K);

    // ---- stage the input tile (zero outside the input rectangle); every load of a thread
    // is issued before its LDS stores so the latencies overlap
    constexpr int NE = (LH * LW0 + NT - 1) / NT;
    T v[NE];
    if constexpr (KIND == CONV_ADJ) {
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = threadIdx.x + NT * q;
            const int ly = e / LW0, lx = e - ly * LW0;
            const int y = iy_base + ly, x = ix_base + lx;
            T val = 0;
            if (e < LH * LW0 && y >= 0 && y < im.H && x >= 0 && x < im.W) {
                // a pixel's seed reaches each of its sub-pixels (the adjoint of their sum)
                const long long pix = im.pix_off + (long long)(y / im.up) * im.Wc + x / im.up;
                val = io.seed ? io.seed[pix] : -2.f * io.weight[pix] * p.rbuf[pix];
            }
            v[q] = val;
        }
    } else {
        const T* __restrict__ in = (jb.in_src ? io.in_s : io.in) + jb.in_off + (long long)it.ch * jb.in_cs;
        const int iy1 = jb.in_y0 + jb.in_h, ix1 = jb.in_x0 + jb.in_w;
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = threadIdx.x + NT * q;
            const int ly = e / LW0, lx = e - ly * LW0;
            const int y = iy_base + ly, x = ix_base + lx;
            T val = 0;
            if (e < LH * LW0 && y >= jb.in_y0 && y < iy1 && x >= jb.in_x0 && x < ix1)
                val = in[(long long)(y - jb.in_y0) * jb.in_w + (x - jb.in_x0)];
            v[q] = val;
        }
    }
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const int e = threadIdx.x + NT * q;
        if (e < LH * LW0) {
            const int ly = e / LW0, lx = e - ly * LW0;
            tile[ly * LW + lx] = v[q];
        }
    }
    __syncthreads();

    // ---- register-window convolution
    const int ty = (int)threadIdx.x / LPR, tx = (int)threadIdx.x % LPR;
    T acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0;
    for (int U = 0; U < P; ++U) {
        const T* row = tile + (ty + P - 1 - U) * LW + tx * R;
        T s[R + P - 1];
#pragma unroll
        for (int k = 0; k < R + P - 1; ++k) s[k] = row[k];
        T part[R];
#pragma unroll
        for (int r = 0; r < R; ++r) part[r] = 0;
#pragma unroll
        for (int V = 0; V < P; ++V) {
            // the PSF value (scalar load) moves from its SGPR into a VGPR, one v_mov per R FMAs:
            // gfx950 issues FMAs of VGPR operands from two waves at once, FMAs that read an
            // SGPR one at a time (measured 124 vs 76 TFLOP/s)
            T kv;
            if constexpr (KLDS) kv = kt[U * KP + V];
            else asm("v_mov_b32 %0, %1" : "=v"(kv) : "s"(K[U * P + V]));
#pragma unroll
            for (int r = 0; r < R; ++r) part[r] = fma(kv, s[r + P - 1 - V], part[r]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += part[r];
    }

    // ---- epilogue
    const int y = oy0 + ty;
    const int xb = ox0 + tx * R;
    const int xend = jb.out_x0 + jb.out_w;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int up = im.up;
    if constexpr (KIND != CONV_ADJ) bin_pixels<LPR>(acc, up);
    const int nq = KIND == CONV_ADJ ? R : R / up;               // values per lane
    const int sx = KIND == CONV_ADJ ? 1 : up;                   // render-grid step between them
    const bool yok = y < jb.out_y0 + jb.out_h && (KIND == CONV_ADJ || (ty & (up - 1)) == 0);
    const int yc = KIND == CONV_ADJ ? y : y / up;               // image pixel row
    if constexpr (KIND == CONV_FWD) {
        fwd_epilogue<T, R, NW>(p, jb, im, io, item_idx, acc, y, xb, yok, red);
    } else if constexpr (KIND == CONV_JCOL) {
        float* __restrict__ out = io.out + jb.out_off + (long long)it.ch * jb.out_cs;
        double s1 = 0.0, s2 = 0.0;
        const bool epart = io.weight && !jb.gram_part;       // sum w r J and sum w J here
        if (yok) {
            // the column's plane is stored on the image pixels of the output box
            const int ow = jb.out_w / up;
            const long long orow = (long long)(yc - jb.out_y0 / up) * ow - jb.out_x0 / up;
            const long long rowpix = im.pix_off + (long long)yc * im.Wc;
            float wv[R], rv[R];                   // loads first, as above
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int x = xb + r * sx;
                wv[r] = rv[r] = 0.f;
                if (epart && r < nq && x < xend) {
                    wv[r] = io.weight[rowpix + x / up];
                    rv[r] = p.rbuf[rowpix + x / up];
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int x = xb + r * sx;
                if (r < nq && x < xend) {
                    const int xc = x / up;
                    out[orow + xc] = acc[r];
                    if (epart) {
                        const double wj = (double)wv[r] * (double)acc[r];
                        s1 += wj * (double)rv[r];
                        s2 += wj;
                    }
                }
            }
        }
        if (epart) {
            s1 = conv_wave_sum(s1);
            s2 = conv_wave_sum(s2);
            if (lane == 0) { red[wv][0] = s1; red[wv][1] = s2; }
            __syncthreads();
            if (threadIdx.x < 2) {
                const int q = threadIdx.x;
                double sum = red[0][q];
#pragma unroll
                for (int w = 1; w < NW; ++w) sum += red[w][q];
                io.part[(long long)item_idx * 2 + q] = sum;
            }
        }
    } else {
        float* __restrict__ out = io.out + jb.out_off;
        if (yok) {
            const long long orow = (long long)(y - jb.out_y0) * jb.out_w - jb.out_x0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int x = xb + r;
                if (x < xend) out[orow + x] = acc[r];
            }
        }
    }
}

// Row pitch (in doubles) of the FP64 kernel's LDS tile: an odd number of 16-byte chunks.  The
// lanes of one output row read windows 64 bytes apart (every fourth bank group); with an even
// number of chunks the rows of a wave fall on the same groups (P = 25, 2048 x 2048: 109 us at
// a pitch of 88 doubles, 70 us at 90; P = 15: 51 us at 80, 34 us at 78).
constexpr int pitch64(int w) {
    const int e = (w + 1) & ~1;
    return (e / 2) % 2 ? e : e + 2;
}

// The FP64 objective's model convolution.  Where the stamp is the same upside down (any stamp
// sampled from a round profile; psf_sym, found per call by k_prep), rows U and P - 1 - U
// of the stamp multiply the sum of two input rows: R + P - 1 additions replace P R FMAs.  The
// evaluations of an LM fit (io.fit) take the rows one by one: the fold rounds differently, and a
// fit follows the last bits of its residuals (see k_render64).
// Each window goes through registers in pieces of CH64 taps, the next piece's LDS reads in
// flight while the current one is multiplied.  Above P = 41 the pieces of folded rows are pinned
// in that order (the compiler otherwise reads whole windows of both rows first, 256 registers and
// spills at P = 51: 411 us for 2048 x 2048 against 297 pinned); below, its own order is as fast on
// a full chip and better with one workgroup per CU (P = 31: 35 against 43 us).  Single rows keep
// the compiler's order at every P (pinned 443 against 404 us at P = 51, 891 against 642 at 57).
// Bound by FP64 issue and LDS reads alike: one 2048 x 2048 image, 2 P^2 per output, row by row
// and folded: 36 and 46 TFLOP/s at P = 15, 48 and 67 at P = 25, 51 and 78 at P = 41, 54 and 78 at
// P = 51, 37 and 59 at P = 63 (2-D windows held whole, without a fold: 31, 43, 50, 53, 33).
constexpr int CH64 = 8;
__device__ __forceinline__ void pin(double (&a)[CV_R], int& o1, int& o2) {
    asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]),
                      "+v"(o1), "+v"(o2));
}
__device__ __forceinline__ void pin(double (&a)[CV_R_FINE], int& o1, int& o2) {
    asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(o1), "+v"(o2));
}
template <int P, int TH, int TW, int R>
__global__ __launch_bounds__(TH * TW / R) void k_conv64(PlanPtr pp, const ConvJob* __restrict__ jobs,
                                                        const ConvItem* __restrict__ items, int item_begin,
                                                        ConvIO io) {
    PlanRef p = *pp;
    constexpr int c = (P - 1) / 2;
    constexpr int NT = TH * TW / R;
    constexpr int LPR = TW / R;
    constexpr int NW = NT / 64;
    static_assert(NW >= 1 && NT % 64 == 0, "whole waves");
    constexpr int LH = TH + P - 1;
    constexpr int LW0 = TW + P - 1;
    constexpr int LW = pitch64(LW0);
    __shared__ __attribute__((aligned(16))) double tile[LH * LW];
    __shared__ double red[NW][3];
    constexpr bool KLDS = R != CV_R;
    constexpr int KP = (P + 1) & ~1;
    __shared__ __attribute__((aligned(16))) double kt[KLDS ? P * KP : 1];

    const int item_idx = item_begin + xcd_chunk_item((int)blockIdx.x, (int)gridDim.x);
    const ConvItem it = items[item_idx];
    const ConvJob jb = jobs[it.job];
    const DImage& im = p.images[jb.image];
    if (conv_skipped(p, io, im.sub)) return;
    const int oy0 = jb.out_y0 + it.ty * TH;
    const int ox0 = jb.out_x0 + it.tx * TW;
    const int iy_base = oy0 - c, ix_base = ox0 - c;

    // the stamp does not change during the launch: scalar loads, which the barriers would
    // otherwise turn into vector loads
    using Const = const __attribute__((address_space(4))) double*;
    const Const K = (Const)(p.psf64 + im.psf_off);
    if constexpr (KLDS) stage_stamp<P, KP, NT>(kt, p.psf64 + im.psf_off);

    // ---- stage the input tile (zero outside the input rectangle), NB loads of a thread at a
    // time before their LDS stores
    constexpr int NE = (LH * LW0 + NT - 1) / NT, NB = NE < 24 ? NE : 24;
    {
        const double* __restrict__ in = io.in64 + jb.in_off + (long long)it.ch * jb.in_cs;
        const int iy1 = jb.in_y0 + jb.in_h, ix1 = jb.in_x0 + jb.in_w;
        for (int q0 = 0; q0 < NE; q0 += NB) {
            double v[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int e = (int)threadIdx.x + NT * (q0 + q);
                const int ly = e / LW0, lx = e - ly * LW0;
                const int y = iy_base + ly, x = ix_base + lx;
                v[q] = 0.0;
                if (e < LH * LW0 && y >= jb.in_y0 && y < iy1 && x >= jb.in_x0 && x < ix1)
                    v[q] = in[(long long)(y - jb.in_y0) * jb.in_w + (x - jb.in_x0)];
            }
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int e = (int)threadIdx.x + NT * (q0 + q);
                if (e < LH * LW0) {
                    const int ly = e / LW0, lx = e - ly * LW0;
                    tile[ly * LW + lx] = v[q];
                }
            }
        }
    }
    __syncthreads();

    // ---- register-window convolution
    const int ty = (int)threadIdx.x / LPR, tx = (int)threadIdx.x % LPR;
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
    constexpr int N = R + P - 1, NC = (P + CH64 - 1) / CH64;
    constexpr bool PINNED = P > (R == CV_R ? 41 : 51);           // folded rows
    // acc[r] += sum_V K[U, V] s[r + P - 1 - V], V ascending, s the window that starts at pair o1 of
    // the tile (with TWO: plus the one at pair o2), read from its end as pairs (ds_read_b128).
    // pin() keeps the pieces apart (folded rows): a piece's FMAs come before it, the reads that follow (whose
    // offsets pass through it) after.
    static_assert(N % 2 == 0 && R % 2 == 0 && P % 2 == 1 && LW % 2 == 0 && CH64 % 2 == 0, "windows are whole pairs");
    const double2* tile2 = reinterpret_cast<const double2*>(tile);
    auto row = [&](auto two, int o1, int o2, int U) {
        constexpr bool TWO = decltype(two)::value;
        double s[N], part[R];
        double2 a[CH64 / 2], b[CH64 / 2];
#pragma unroll
        for (int r = 0; r < R; ++r) part[r] = 0.0;
#pragma unroll
        for (int k = P - 1; k < N; k += 2) {
            double2 v = tile2[o1 + k / 2];
            if constexpr (TWO) {
                const double2 w = tile2[o2 + k / 2];
                v.x += w.x;
                v.y += w.y;
            }
            s[k] = v.x;
            s[k + 1] = v.y;
        }
        // entry m below those is s[P - 2 - m]; pairs (m + 1, m), m even
#pragma unroll
        for (int q = 0; q < CH64; q += 2)
            if (q < P - 1) {
                a[q / 2] = tile2[o1 + (P - 3 - q) / 2];
                if constexpr (TWO) b[q / 2] = tile2[o2 + (P - 3 - q) / 2];
            }
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {
#pragma unroll
            for (int q = 0; q < CH64; q += 2) {
                const int m = ch * CH64 + q;
                if (m < P - 1) {
                    s[P - 3 - m] = a[q / 2].x;
                    s[P - 2 - m] = a[q / 2].y;
                    if constexpr (TWO) {
                        s[P - 3 - m] += b[q / 2].x;
                        s[P - 2 - m] += b[q / 2].y;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < CH64; q += 2) {
                const int m = (ch + 1) * CH64 + q;
                if (m < P - 1) {
                    a[q / 2] = tile2[o1 + (P - 3 - m) / 2];
                    if constexpr (TWO) b[q / 2] = tile2[o2 + (P - 3 - m) / 2];
                }
            }
#pragma unroll
            for (int q = 0; q < CH64; ++q) {
                const int V = ch * CH64 + q;
                if (V < P) {
                    double kv;
                    if constexpr (KLDS) kv = kt[U * KP + V];
                    else kv = K[U * P + V];
#pragma unroll
                    for (int r = 0; r < R; ++r) part[r] = fma(kv, s[r + P - 1 - V], part[r]);
                }
            }
            if constexpr (PINNED && TWO) pin(part, o1, o2);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] += part[r];
    };
    const int o0 = (ty * LW + tx * R) / 2;
    const int npair = !io.fit && p.psf_sym[jb.image] ? c : 0;   // block-uniform
    for (int U = 0; U < npair; ++U) row(std::true_type{}, o0 + (P - 1 - U) * (LW / 2), o0 + U * (LW / 2), U);
    for (int U = npair; U < P - npair; ++U) row(std::false_type{}, o0 + (P - 1 - U) * (LW / 2), o0, U);

    // ---- epilogue
    const int y = oy0 + ty;
    bin_pixels<LPR>(acc, im.up);
    const bool yok = y < jb.out_y0 + jb.out_h && (ty & (im.up - 1)) == 0;
    fwd_epilogue<double, R, NW>(p, jb, im, io, item_idx, acc, y, ox0 + tx * R, yok, red);
}

// Jacobian-column convolution with a rank-one stamp K_UV = a_U b_V (jobs of shape
// SHAPE_SEP) as two 1-D passes over an SEP_TH x SEP_TW output tile, 256 threads: the input
// tile with its P - 1 halo is staged in LDS as for the 2-D kernel; the row pass convolves
// every staged row with b into a second LDS buffer (the tile rows plus the vertical halo);
// the column pass convolves that with a, each lane making CV_R consecutive outputs of one
// column, and the epilogue is that of the 2-D kernel's JCOL (column store, and the FP64
// partials of sum w r J and sum w J per item unless the job's gram_part is set).  2 (P + P (TH + P - 1) / TH) multiply-adds per output
// instead of 2 P^2.
template <int P>
__global__ __launch_bounds__(256) void k_conv_sep(PlanPtr pp, const ConvJob* __restrict__ jobs,
                                                  const ConvItem* __restrict__ items, int item_begin,
                                                  ConvIO io) {
    PlanRef p = *pp;
    constexpr int TH = SEP_TH, TW = SEP_TW, NT = 256;
    constexpr int c = (P - 1) / 2;
    constexpr int LPR = TW / CV_R;                  // lanes per output row
    constexpr int NW = NT / 64;
    static_assert(TH * TW / CV_R == NT && TH == CV_R * (NT / TW), "one lane per CV_R outputs of a column");
    constexpr int LH = TH + P - 1;
    constexpr int LW0 = TW + P - 1;
    constexpr int LW = (LW0 + 3) & ~3;
    __shared__ __attribute__((aligned(16))) float tile[LH * LW];
    __shared__ __attribute__((aligned(16))) float hb[LH * TW];
    __shared__ double red[NW][2];

    const int item_idx = item_begin + xcd_chunk_item((int)blockIdx.x, (int)gridDim.x);
    const ConvItem it = items[item_idx];
    const ConvJob jb = jobs[it.job];
    const DImage& im = p.images[jb.image];
    if (conv_skipped(p, io, im.sub)) return;
    const int oy0 = jb.out_y0 + it.ty * TH;
    const int ox0 = jb.out_x0 + it.tx * TW;
    const int iy_base = oy0 - c, ix_base = ox0 - c;

    // ---- stage the input tile (zero outside the input rectangle)
    constexpr int NE = (LH * LW0 + NT - 1) / NT;
    {
        const float* __restrict__ in = (jb.in_src ? io.in_s : io.in) + jb.in_off + (long long)it.ch * jb.in_cs;
        const int iy1 = jb.in_y0 + jb.in_h, ix1 = jb.in_x0 + jb.in_w;
        float v[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = threadIdx.x + NT * q;
            const int ly = e / LW0, lx = e - ly * LW0;
            const int y = iy_base + ly, x = ix_base + lx;
            float val = 0.f;
            if (e < LH * LW0 && y >= jb.in_y0 && y < iy1 && x >= jb.in_x0 && x < ix1)
                val = in[(long long)(y - jb.in_y0) * jb.in_w + (x - jb.in_x0)];
            v[q] = val;
        }
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = threadIdx.x + NT * q;
            if (e < LH * LW0) {
                const int ly = e / LW0, lx = e - ly * LW0;
                tile[ly * LW + lx] = v[q];
            }
        }
    }
    __syncthreads();

    const float* __restrict__ fa = p.psf_sep + im.sep_off;       // a_U (rows)
    const float* __restrict__ fb = fa + P;                       // b_V (columns)
    // ---- row pass: hb[r][x] = sum_V b_V tile[r][x + P - 1 - V], r < LH, x < TW
    for (int task = (int)threadIdx.x; task < LH * LPR; task += NT) {
        const int r = task / LPR, g = task - r * LPR;
        const float* row = tile + r * LW + g * CV_R;
        float sw[CV_R + P - 1];
#pragma unroll
        for (int k = 0; k < CV_R + P - 1; ++k) sw[k] = row[k];
        float part[CV_R];
#pragma unroll
        for (int q = 0; q < CV_R; ++q) part[q] = 0.f;
#pragma unroll
        for (int V = 0; V < P; ++V) {
            // the factor (a scalar load) moves into a VGPR, one v_mov per CV_R FMAs, so that
            // the FMAs of two waves issue together (as in the 2-D kernel)
            float kv;
            asm("v_mov_b32 %0, %1" : "=v"(kv) : "s"(fb[V]));
#pragma unroll
            for (int q = 0; q < CV_R; ++q) part[q] = fmaf(kv, sw[q + P - 1 - V], part[q]);
        }
#pragma unroll
        for (int q = 0; q < CV_R; ++q) hb[r * TW + g * CV_R + q] = part[q];
    }
    __syncthreads();

    // ---- column pass: out[y][x] = sum_U a_U hb[y + P - 1 - U][x]; each lane makes CV_R
    // consecutive outputs of one column from a register window down that column (lanes of
    // a wave take consecutive columns: conflict-free LDS reads, coalesced stores)
    const int cx = (int)threadIdx.x % TW, rb = (int)threadIdx.x / TW;      // column, row block
    float acc[CV_R];
    {
        float sw[CV_R + P - 1];
#pragma unroll
        for (int k = 0; k < CV_R + P - 1; ++k) sw[k] = hb[(rb * CV_R + k) * TW + cx];
#pragma unroll
        for (int q = 0; q < CV_R; ++q) acc[q] = 0.f;
#pragma unroll
        for (int U = 0; U < P; ++U) {
            float ka;
            asm("v_mov_b32 %0, %1" : "=v"(ka) : "s"(fa[U]));
#pragma unroll
            for (int q = 0; q < CV_R; ++q) acc[q] = fmaf(ka, sw[q + P - 1 - U], acc[q]);
        }
    }

    // ---- epilogue (the JCOL epilogue of the 2-D kernel on a pixel grid)
    const int x = ox0 + cx;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float* __restrict__ out = io.out + jb.out_off + (long long)it.ch * jb.out_cs;
    double s1 = 0.0, s2 = 0.0;
    const bool epart = io.weight && !jb.gram_part;           // sum w r J and sum w J here
    if (x < jb.out_x0 + jb.out_w) {
        // the column's weights and residuals first: their loads overlap instead of following
        // one another
        float wv[CV_R], rv[CV_R];
#pragma unroll
        for (int q = 0; q < CV_R; ++q) {
            const int y = oy0 + rb * CV_R + q;
            wv[q] = rv[q] = 0.f;
            if (epart && y < jb.out_y0 + jb.out_h) {
                const long long pix = im.pix_off + (long long)y * im.Wc + x;
                wv[q] = io.weight[pix];
                rv[q] = p.rbuf[pix];
            }
        }
#pragma unroll
        for (int q = 0; q < CV_R; ++q) {
            const int y = oy0 + rb * CV_R + q;
            if (y < jb.out_y0 + jb.out_h) {
                out[(long long)(y - jb.out_y0) * jb.out_w + (x - jb.out_x0)] = acc[q];
                if (epart) {
                    const double wj = (double)wv[q] * (double)acc[q];
                    s1 += wj * (double)rv[q];
                    s2 += wj;
                }
            }
        }
    }
    if (epart) {
        s1 = conv_wave_sum(s1);
        s2 = conv_wave_sum(s2);
        if (lane == 0) { red[wv][0] = s1; red[wv][1] = s2; }
        __syncthreads();
        if (threadIdx.x < 2) {
            const int q = threadIdx.x;
            double sum = red[0][q];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += red[w][q];
            io.part[(long long)item_idx * 2 + q] = sum;
        }
    }
}

#define APX_FOR_EACH_P(X)                                                                     \
    X(1) X(3) X(5) X(7) X(9) X(11) X(13) X(15) X(17) X(19) X(21) X(23) X(25) X(27) X(29)     \
    X(31) X(33) X(35) X(37) X(39) X(41) X(43) X(45) X(47) X(49) X(51) X(53) X(55) X(57)      \
    X(59) X(61) X(63)

template <int KIND, typename T, int TH, int TW, int R>
hipError_t launch_conv_shape(const Plan& p, const ConvLaunch& L, const ConvIO& io, hipStream_t st) {
    dim3 grid(L.item_count), block(TH * TW / R);
    switch (L.P) {
#define APX_CASE(PP)                                                                                     \
    case PP:                                                                                             \
        if constexpr (sizeof(T) == 8)                                                                    \
            hipLaunchKernelGGL((k_conv64<PP, TH, TW, R>), grid, block, 0, st, p.dev, L.jobs, L.items,        \
                               L.item_begin, io);                                                        \
        else                                                                                             \
            hipLaunchKernelGGL((k_conv<PP, KIND, TH, TW, R>), grid, block, 0, st, p.dev, L.jobs, L.items,    \
                               L.item_begin, io);                                                        \
        break;
        APX_FOR_EACH_P(APX_CASE)
#undef APX_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

inline hipError_t launch_conv_sep_impl(const Plan& p, const ConvLaunch& L, const ConvIO& io, hipStream_t st) {
    if (L.item_count <= 0) return hipSuccess;
    dim3 grid(L.item_count), block(256);
    switch (L.P) {
#define APX_CASE(PP)                                                                                   \
    case PP:                                                                                           \
        hipLaunchKernelGGL((k_conv_sep<PP>), grid, block, 0, st, p.dev, L.jobs, L.items, L.item_begin, io); \
        break;
        APX_FOR_EACH_P(APX_CASE)
#undef APX_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int KIND, typename T = float>
hipError_t launch_conv_kind(const Plan& p, const ConvLaunch& L, const ConvIO& io, hipStream_t st) {
    if (L.item_count <= 0) return hipSuccess;
    static_assert(N_TILE_SHAPES == 4, "one case per tile shape");
    switch (L.shape) {
        case 0: return launch_conv_shape<KIND, T, tile_th(0), tile_tw(0), CV_R>(p, L, io, st);
        case 1: return launch_conv_shape<KIND, T, tile_th(1), tile_tw(1), CV_R>(p, L, io, st);
        case 2: return launch_conv_shape<KIND, T, tile_th(2), tile_tw(2), CV_R>(p, L, io, st);
        case FINE_SHAPE:
            if (L.fine) return launch_conv_shape<KIND, T, tile_th(FINE_SHAPE), tile_tw(FINE_SHAPE), CV_R_FINE>(p, L, io, st);
            return launch_conv_shape<KIND, T, tile_th(FINE_SHAPE), tile_tw(FINE_SHAPE), CV_R>(p, L, io, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace apx
