// Normal-equation kernels: J^T W J tiles on FP64 MFMA, ordered reductions and the
// assembly of J^T W J, J^T W r, chi^2 and the gradient from their partial sums.
//
// A_pq = sum_i w_i J_ip J_iq (§2.5, the Gauss-Newton Hessian of Eq. chi2).  Columns of
// one group share an output box; the product of two groups runs over the intersection
// of their boxes.  FP32 Jacobian entries are promoted to FP64 (w J_p is exact in FP64) and
// contracted on FP64 MFMA: 64 x 64 tiles staged in LDS for two wide groups, 4 x 4 blocks
// straight from registers for the others.  Every tile of every slice of pixels is written to
// its own slot and summed later in a fixed order, so the result does not depend on scheduling.
#include <type_traits>

#include "apx_internal.h"
#include "lm_state.h"

namespace apx {

typedef double apx_d4 __attribute__((ext_vector_type(4)));

// Two wide groups, 64 x 64 tiles: the tile's 16 x 16 blocks that hold needed entries (a block
// is skipped when its rows or its columns lie past the group's last column, or, on a diagonal
// tile of a group with itself, when it lies wholly below the diagonal) are dealt to the 4 waves
// in turn, at most 4 blocks (MFMA accumulators) each.
// Stages of KC = PAIR_KC pixels (one row segment of the box intersection) are software
// pipelined two deep: the global loads of stages s+1 and s+2 are in flight while the
// MFMAs consume s.  Each thread stages the same tile columns and pixel offsets in every
// stage, so its column offsets into J are computed once.
__global__ __launch_bounds__(256) void k_pair(PlanPtr pp, const DPair* __restrict__ pairs,
                                              const PairItem* __restrict__ items,
                                              const float* __restrict__ weight,
                                              const apx_lm_state* lm) {
    PlanRef p = *pp;
    constexpr int KC = PAIR_KC, TM = 64;
    constexpr int PER = TM * KC / 256;              // elements of A (and of B) per thread
    constexpr int NB = 2;                           // accumulators: NB x NB per wave
    __shared__ double As[TM][KC + 1];
    __shared__ double Bs[TM][KC + 1];
    // the 64-wide tile pairs of one K-slice (up to 21 for a 350-column group) share its rows
    // of J in one L2 when each XCD takes a contiguous range of items (in runs of 8 they read
    // J 3.3x over from HBM)
    const PairItem it = items[xcd_item((int)blockIdx.x, (int)gridDim.x)];
    const DPair pr = pairs[it.pair];
    if (lm && lm[pr.sub].need_jac == 0) return;
    // by value: the fields live in registers for the whole loop (no reloads through the
    // pointers after every store)
    const DGroup G = p.groups[pr.g];
    const DGroup Hh = p.groups[pr.h];
    const long long pix_off = p.images[pr.image].pix_off;
    const int imW = p.images[pr.image].Wc;          // image pixels (output boxes are in pixels)
    const long long gs = (long long)G.oh * G.ow, hs = (long long)Hh.oh * Hh.ow;
    const float* __restrict__ Jg = p.J + G.j_off;
    const float* __restrict__ Jh = p.J + Hh.j_off;
    const int a0 = it.ta * TM, b0 = it.tb * TM;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // this wave's blocks s < nbk, row block (blk >> 4 s) & 3, column block
    // (blk >> (4 s + 2)) & 3
    int blk = 0, nbk = 0;
    {
        const int rows = G.ncols - a0, cols = Hh.ncols - b0;
        const bool diag = pr.g == pr.h && it.ta == it.tb;
        int k = 0;
        for (int m = 0; m < 4; ++m)
            for (int n = 0; n < 4; ++n) {
                if (16 * m >= rows || 16 * n >= cols || (diag && m > n)) continue;
                if ((k & 3) == wv) {
                    blk |= (m | (n << 2)) << (4 * nbk);
                    ++nbk;
                }
                ++k;
            }
    }
    auto bm = [&](int q) { return (blk >> (4 * q)) & 3; };
    auto bn = [&](int q) { return (blk >> (4 * q + 2)) & 3; };
    apx_d4 acc[NB][NB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = (apx_d4){0.0, 0.0, 0.0, 0.0};

    // element q of this thread: tile column i0 + DI q at stage pixel kq, the same in every
    // stage; its offset into J is colA + q * stepA (the step is uniform)
    constexpr int DI = 256 / KC;
    const int i0 = threadIdx.x / KC, kq = threadIdx.x % KC;
    const long long colA = (long long)(a0 + i0) * gs - G.ox0, stepA = (long long)DI * gs;
    const long long colB = (long long)(b0 + i0) * hs - Hh.ox0, stepB = (long long)DI * hs;
    const int nva = G.ncols - a0 - i0, nvb = Hh.ncols - b0 - i0;   // element q valid: DI q < nv
    const long long lastA = (long long)(G.ncols - 1) * gs - G.ox0;   // a column that exists
    const long long lastB = (long long)(Hh.ncols - 1) * hs - Hh.ox0;

    const int nxs = (pr.x1 - pr.x0 + KC - 1) / KC;
    const int n_stage = it.s1 - it.s0;
    // two stages of global loads in flight (register ring): the loads of stage s+2 are
    // issued while the MFMAs consume stages s and s+1
    float ra0[PER], rb0[PER], rw0 = 0.f, ra1[PER], rb1[PER], rw1 = 0.f;
    // every load is issued unconditionally (a lane past the box or past the last column
    // reads a valid entry and zeroes it afterwards), so the 2 PER + 1 loads of a stage go
    // out back to back instead of one branch each
    auto fetch = [&](int st, float (&ra)[PER], float (&rb)[PER], float& rw) {
        const int gs_ = it.s0 + st;
        const int row = pr.y0 + gs_ / nxs;
        const int x = pr.x0 + (gs_ - (gs_ / nxs) * nxs) * KC + kq;
        const bool in = x < pr.x1;
        const int xc = in ? x : pr.x1 - 1;
        const long long grow = (long long)(row - G.oy0) * G.ow + xc;
        const long long hrow = (long long)(row - Hh.oy0) * Hh.ow + xc;
        const float wv = weight[pix_off + (long long)row * imW + xc];
        rw = in ? wv : 0.f;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const bool va = DI * q < nva, vb = DI * q < nvb;
            const float a = Jg[(va ? colA + q * stepA : lastA) + grow];
            const float b = Jh[(vb ? colB + q * stepB : lastB) + hrow];
            ra[q] = (in && va) ? a : 0.f;
            rb[q] = (in && vb) ? b : 0.f;
        }
    };
    auto stage = [&](const float (&ra)[PER], const float (&rb)[PER], float rw) {
        const double wd = (double)rw;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            As[i0 + DI * q][kq] = (double)ra[q] * wd;
            Bs[i0 + DI * q][kq] = (double)rb[q];
        }
    };
    auto compute = [&]() {
        // one branch per stage on the wave's block count; inside, the LDS reads of a
        // K step are all issued before its MFMAs
        // a wave with fewer than 4 blocks spreads each over 4 / NS accumulators (K steps
        // dealt in turn), so it still has 4 independent MFMA chains
        auto run = [&](auto ns) {
            constexpr int NS = decltype(ns)::value;
            constexpr int R = NS == 1 ? 4 : NS == 2 ? 2 : 1;
#pragma unroll
            for (int kk = 0; kk < KC; kk += 4) {
                const int rr = (kk / 4) % R;
                double av[NS], bv[NS];
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    av[q] = As[bm(q) * 16 + (lane & 15)][kk + (lane >> 4)];
                    bv[q] = Bs[bn(q) * 16 + (lane & 15)][kk + (lane >> 4)];
                }
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    const int c = q * R + rr;
                    acc[c >> 1][c & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q], bv[q], acc[c >> 1][c & 1], 0, 0, 0);
                }
            }
        };
        switch (nbk) {
            case 4: run(std::integral_constant<int, 4>{}); break;
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 2: run(std::integral_constant<int, 2>{}); break;
            case 1: run(std::integral_constant<int, 1>{}); break;
            default: break;
        }
    };
    if (n_stage > 0) fetch(0, ra0, rb0, rw0);
    if (n_stage > 1) fetch(1, ra1, rb1, rw1);
    for (int st = 0; st < n_stage; st += 2) {
        stage(ra0, rb0, rw0);
        __syncthreads();
        if (st + 2 < n_stage) fetch(st + 2, ra0, rb0, rw0);
        compute();
        __syncthreads();
        if (st + 1 < n_stage) {
            stage(ra1, rb1, rw1);
            __syncthreads();
            if (st + 3 < n_stage) fetch(st + 3, ra1, rb1, rw1);
            compute();
            __syncthreads();
        }
    }

    double* out = p.pair_part + it.out_off;
    // blocks no wave holds are left unwritten: the assembly reads none of their entries.
    // A block's R accumulators are added in order.
    auto emit = [&](auto ns) {
        constexpr int NS = decltype(ns)::value;
        constexpr int R = NS == 1 ? 4 : NS == 2 ? 2 : 1;
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double sum = acc[(q * R) >> 1][(q * R) & 1][v];
#pragma unroll
                for (int r = 1; r < R; ++r) sum += acc[(q * R + r) >> 1][(q * R + r) & 1][v];
                // v_mfma_f64_16x16x4: D[i][j] sits in lane j + 16 (i % 4), register i / 4
                const int i = bm(q) * 16 + (lane >> 4) + 4 * v;
                const int j = bn(q) * 16 + (lane & 15);
                out[i * TM + j] = sum;
            }
    };
    switch (nbk) {
        case 4: emit(std::integral_constant<int, 4>{}); break;
        case 3: emit(std::integral_constant<int, 3>{}); break;
        case 2: emit(std::integral_constant<int, 2>{}); break;
        case 1: emit(std::integral_constant<int, 1>{}); break;
        default: break;
    }
}

// J^T W J of narrow column groups on v_mfma_f64_4x4x4f64: the instruction holds four
// independent 4 x 4 x 4 products (blocks), block b of lanes 16 k + 4 b + i (A[i][k], B[k][j] at
// lane 16 k + 4 b + j, D[i][j] at lane 16 i + 4 b + j; measured on gfx950).  Lane L takes pixel
// L / 4 of a 16-pixel chunk and column L % 4 of a tile of 4 columns, so one instruction
// contracts 16 pixels of one 4 x 4 tile pair, and the tiles are loaded straight from J into
// registers (each reused by every pair it is in).  The items of a group with itself (k_gram4) are
// stages of PAIR_KC pixels of a row, padded at row ends; those of two groups (k_cross4) are runs
// of pixels counted along the rows of the pair's box (no padding).  The row of a stage or of a
// pixel comes from a multiplication by the reciprocal of the row's length (GramDiv).  All loads
// of a wave's next chunks are issued before the MFMAs of the current ones.  At the end each wave
// folds its four blocks (lanes xor 4, xor 8) and the four waves are added in order.
// What bounds them: latency of the loads while there are few waves (k_cross4's runs are cut
// short enough to fill the chip, add_runs in the plan), then for wide groups the MFMAs (35
// columns: 54 per 16 pixels, 98 us of MFMA issue in the 192 us that 3.9 M pixels take in
// k_gram4) and for narrow ones the loads (8 columns against 8, 28 M pixels: 273 us).
struct GramDiv {                                    // e / bw for 0 <= e < 2^31, bw >= 1
    unsigned m, bw;                                 // m = floor((2^32 - 1) / bw)
    __device__ __forceinline__ explicit GramDiv(int w) : m(0xffffffffu / (unsigned)w), bw((unsigned)w) {}
    __device__ __forceinline__ void operator()(int e, int& row, int& x) const {
        unsigned q = __umulhi((unsigned)e, m);       // the quotient or one less
        unsigned r = (unsigned)e - q * bw;
        if (r >= bw) { r -= bw; ++q; }
        row = (int)q;
        x = (int)r;
    }
};

// The per-wave sums of NQ blocks: folded over the four blocks of the instruction, then over the
// four waves in order, into out[NQ * 16] (block q: entry (i, j) at 16 q + 4 i + j).
template <int NQ>
__device__ __forceinline__ void gram_emit(const double (&acc)[NQ], double* __restrict__ out) {
    __shared__ double red[4][NQ * 16];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double v = acc[q];
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 8, 64);
        // lanes with block 0 (lane % 16 < 4) hold D[i][j] at lane 16 i + j
        if ((lane & 12) == 0) red[wv][q * 16 + (lane >> 4) * 4 + (lane & 3)] = v;
    }
    __syncthreads();
    for (int e = (int)threadIdx.x; e < NQ * 16; e += 256)
        out[e] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
}

// A group (NT tiles of 4 columns, at most 36 columns) with itself: every tile pair a <= b, and
// each tile against [r 1 0 0] (the pixel's residual, a one), which gives the columns' J^T W r
// and sum w J (the sky row of J^T W J) over the item in NT more blocks after the tile pairs.
// Its items are up to 128 stages of PAIR_KC pixels of a row (stage s: row s / nxs of the box,
// pixels (s % nxs) PAIR_KC ..., nxs stages a row), wave w taking stages s0 + w, + 4, ... in
// order: the order of these sums is part of a fit's result (its later steps follow the last
// bits of this one through the FP32 derivative images), so it does not follow the number of
// items of a launch.  NS chunks of 16 pixels of a wave are in flight.
template <int NT, int NS>
__global__ __launch_bounds__(256) void k_gram4(PlanPtr pp, const DPair* __restrict__ pairs,
                                               const PairItem* __restrict__ items, int n_items,
                                               const float* __restrict__ weight, const apx_lm_state* lm) {
    PlanRef p = *pp;
    constexpr int NP = NT * (NT + 1) / 2, NH = PAIR_KC / 16;     // chunks of a stage
    static_assert(NS % NH == 0, "whole stages in flight");
    const PairItem it = items[xcd_chunk_item((int)blockIdx.x, n_items)];
    const DPair pr = pairs[it.pair];
    if (lm && lm[pr.sub].need_jac == 0) return;
    const DGroup G = p.groups[pr.g];
    const int imW = p.images[pr.image].Wc, bw = pr.x1 - pr.x0;
    const long long gs = (long long)G.oh * G.ow;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 3, pxl = lane >> 2;       // column within a tile, pixel within a chunk
    const float* __restrict__ Jg = p.J + G.j_off + (long long)(pr.y0 - G.oy0) * G.ow + (pr.x0 - G.ox0);
    const long long pix0 = p.images[pr.image].pix_off + (long long)pr.y0 * imW + pr.x0;
    const float* __restrict__ wb = weight + pix0;
    const float* __restrict__ rb = p.rbuf + pix0;
    const GramDiv div((bw + PAIR_KC - 1) / PAIR_KC);
    const float* cb[NT];                             // this lane's column of each tile
    bool cval[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int ca = 4 * t + col;
        cval[t] = ca < G.ncols;
        cb[t] = Jg + (long long)(cval[t] ? ca : G.ncols - 1) * gs;
    }
    double acc[NP + NT];
#pragma unroll
    for (int q = 0; q < NP + NT; ++q) acc[q] = 0.0;
    auto fetch = [&](int st0, float (&bv)[NS][NT], float (&wf)[NS], float (&rf)[NS], bool (&in)[NS]) {
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const int st = st0 + 4 * (h / NH);
            int row, sx;
            div(st < it.s1 ? st : it.s1 - 1, row, sx);
            const int x = sx * PAIR_KC + 16 * (h % NH) + pxl;
            in[h] = st < it.s1 && x < bw;
            const int xc = x < bw ? x : bw - 1;
            const long long pix = (long long)row * imW + xc, grow = (long long)row * G.ow + xc;
            wf[h] = wb[pix];
            rf[h] = rb[pix];
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[h][t] = cb[t][grow];
        }
    };
    float bc[NS][NT], wc[NS], rc[NS];
    bool ic[NS];
    int st = it.s0 + wv;
    if (st < it.s1) fetch(st, bc, wc, rc, ic);
    while (st < it.s1) {
        const int st1 = st + 4 * (NS / NH);
        float bn[NS][NT], wn[NS], rn[NS];
        bool in[NS];
        const bool more = st1 < it.s1;
        if (more) fetch(st1, bn, wn, rn, in);
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const double w = ic[h] ? (double)wc[h] : 0.0;
            const double vx = col == 0 ? (double)rc[h] : (col == 1 ? 1.0 : 0.0);     // [r 1 0 0]
            double b[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) b[t] = (ic[h] && cval[t]) ? (double)bc[h][t] : 0.0;
            int q = 0;
#pragma unroll
            for (int ta = 0; ta < NT; ++ta) {
                const double a = b[ta] * w;
#pragma unroll
                for (int tb = ta; tb < NT; ++tb, ++q)
                    acc[q] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b[tb], acc[q], 0, 0, 0);
                acc[NP + ta] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, vx, acc[NP + ta], 0, 0, 0);
            }
        }
        if (more) {
#pragma unroll
            for (int h = 0; h < NS; ++h) {
#pragma unroll
                for (int t = 0; t < NT; ++t) bc[h][t] = bn[h][t];
                wc[h] = wn[h];
                rc[h] = rn[h];
                ic[h] = in[h];
            }
        }
        st = st1;
    }
    gram_emit<NP + NT>(acc, p.pair_part + it.out_off);
}

// Two groups of which at least one is narrow: BA tiles of 4 columns of pr.g against BB tiles
// of pr.h over the item's pixels (tile columns past a group's last read it and count as zero).
// (On 16 x 16 MFMA tiles two 7-column galaxies filled 49 of 256 entries: the overlaps of 60
// galaxies on four 700 x 700 images took 562 us there, 273 us here.)
template <int BA, int BB>
__global__ __launch_bounds__(256) void k_cross4(PlanPtr pp, const DPair* __restrict__ pairs,
                                                const PairItem* __restrict__ items, int n_items,
                                                const float* __restrict__ weight, const apx_lm_state* lm) {
    PlanRef p = *pp;
    constexpr int NS = BA + BB <= 4 ? 4 : 2;
    const PairItem it = items[xcd_chunk_item((int)blockIdx.x, n_items)];
    const DPair pr = pairs[it.pair];
    if (lm && lm[pr.sub].need_jac == 0) return;
    const DGroup G = p.groups[pr.g];
    const DGroup Hh = p.groups[pr.h];
    const int imW = p.images[pr.image].Wc;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 3, pxl = lane >> 2;
    const int yb = pr.y0 + it.row0;
    const float* __restrict__ Jg = p.J + G.j_off + (long long)(yb - G.oy0) * G.ow + (pr.x0 - G.ox0);
    const float* __restrict__ Jh = p.J + Hh.j_off + (long long)(yb - Hh.oy0) * Hh.ow + (pr.x0 - Hh.ox0);
    const float* __restrict__ wb = weight + p.images[pr.image].pix_off + (long long)yb * imW + pr.x0;
    const GramDiv div(pr.x1 - pr.x0);
    const float *ca[BA], *cb[BB];
    bool va[BA], vb[BB];
#pragma unroll
    for (int t = 0; t < BA; ++t) {
        const int c = 4 * (it.ta + t) + col;
        va[t] = c < G.ncols;
        ca[t] = Jg + (long long)(va[t] ? c : G.ncols - 1) * G.oh * G.ow;
    }
#pragma unroll
    for (int t = 0; t < BB; ++t) {
        const int c = 4 * (it.tb + t) + col;
        vb[t] = c < Hh.ncols;
        cb[t] = Jh + (long long)(vb[t] ? c : Hh.ncols - 1) * Hh.oh * Hh.ow;
    }
    double acc[BA * BB];
#pragma unroll
    for (int q = 0; q < BA * BB; ++q) acc[q] = 0.0;
    auto fetch = [&](int e0, float (&av)[NS][BA], float (&bv)[NS][BB], float (&wf)[NS]) {
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const int e = e0 + 16 * h + pxl;
            const bool in = e < it.s1;
            int row, x;
            div(in ? e : it.s1 - 1, row, x);
            const long long grow = (long long)row * G.ow + x, hrow = (long long)row * Hh.ow + x;
            const float wl = wb[(long long)row * imW + x];
#pragma unroll
            for (int t = 0; t < BA; ++t) av[h][t] = ca[t][grow];
#pragma unroll
            for (int t = 0; t < BB; ++t) bv[h][t] = cb[t][hrow];
            wf[h] = in ? wl : 0.f;
        }
    };
    float ac[NS][BA], bc[NS][BB], wc[NS];
    int e0 = it.s0 + 16 * NS * wv;
    if (e0 < it.s1) fetch(e0, ac, bc, wc);
    while (e0 < it.s1) {
        const int e1 = e0 + 64 * NS;
        float an[NS][BA], bn[NS][BB], wn[NS];
        const bool more = e1 < it.s1;
        if (more) fetch(e1, an, bn, wn);
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const bool in = e0 + 16 * h + pxl < it.s1;
            const double w = (double)wc[h];
            double a[BA], b[BB];
#pragma unroll
            for (int t = 0; t < BA; ++t) a[t] = (in && va[t]) ? (double)ac[h][t] * w : 0.0;
#pragma unroll
            for (int t = 0; t < BB; ++t) b[t] = (in && vb[t]) ? (double)bc[h][t] : 0.0;
#pragma unroll
            for (int ta = 0; ta < BA; ++ta)
#pragma unroll
                for (int tb = 0; tb < BB; ++tb)
                    acc[ta * BB + tb] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[ta], b[tb], acc[ta * BB + tb], 0, 0, 0);
        }
        if (more) {
#pragma unroll
            for (int h = 0; h < NS; ++h) {
#pragma unroll
                for (int t = 0; t < BA; ++t) ac[h][t] = an[h][t];
#pragma unroll
                for (int t = 0; t < BB; ++t) bc[h][t] = bn[h][t];
                wc[h] = wn[h];
            }
        }
        e0 = e1;
    }
    gram_emit<BA * BB>(acc, p.pair_part + it.out_off);
}

hipError_t launch_gram4(const Plan& p, const PairLaunch& L, const float* weight,
                        const apx_lm_state* lm, hipStream_t st) {
    if (L.n_items <= 0) return hipSuccess;
    dim3 grid(L.n_items), block(256);
    switch (L.tm) {
#define APX_G4(T)                                                                                       \
    case T:                                                                                             \
        hipLaunchKernelGGL((k_gram4<T, (T) <= 2 ? 8 : (T) <= 5 ? 4 : 2>), grid, block, 0, st, p.dev, L.pairs, L.items, L.n_items, weight, lm); \
        break;
        APX_G4(1) APX_G4(2) APX_G4(3) APX_G4(4) APX_G4(5) APX_G4(6) APX_G4(7) APX_G4(8) APX_G4(9)
#undef APX_G4
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_cross4(const Plan& p, const PairLaunch& L, const float* weight,
                         const apx_lm_state* lm, hipStream_t st) {
    if (L.n_items <= 0) return hipSuccess;
    dim3 grid(L.n_items), block(256);
    static_assert(N_CROSS == 9, "one case per block shape");
    switch (L.tm) {
#define APX_X4(K)                                                                                              \
    case K:                                                                                                    \
        hipLaunchKernelGGL((k_cross4<cross_a(K), cross_b(K)>), grid, block, 0, st, p.dev, L.pairs, L.items, L.n_items, \
                           weight, lm);                                                                        \
        break;
        APX_X4(0) APX_X4(1) APX_X4(2) APX_X4(3) APX_X4(4) APX_X4(5) APX_X4(6) APX_X4(7) APX_X4(8)
#undef APX_X4
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int pair_blocks_per_cu() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_pair, 256, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return nb;
}

hipError_t launch_pairs(const Plan& p, const PairLaunch& L, const float* weight,
                        const apx_lm_state* lm, hipStream_t st) {
    if (L.n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pair, dim3(L.n_items), dim3(256), 0, st, p.dev, L.pairs, L.items, weight, lm);
    return hipGetLastError();
}

// Sum over entries b + lane, b + lane + 64, ... < e of load(k), four loads of a lane in flight:
// the same order on every run.
template <class F>
__device__ __forceinline__ double lane_sum(int b, int e, F&& load) {
    double acc = 0.0;
    for (int k = b + (int)(threadIdx.x & 63); k < e; k += 256) {
        double v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = k + 64 * q < e ? load(k + 64 * q) : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc += v[q];
    }
    return acc;
}
__device__ __forceinline__ double butterfly(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// One wave per (column, component).
__global__ __launch_bounds__(256) void k_col_sums(PlanPtr pp, const int* __restrict__ col_seg,
                                                  const int* __restrict__ col_idx) {
    PlanRef p = *pp;
    const int sf = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (sf >= 2 * p.n_cols) return;
    const int c = sf >> 1, q = sf & 1;
    const double v = butterfly(lane_sum(col_seg[c], col_seg[c + 1], [&](int k) { return p.jcol_part[2LL * col_idx[k] + q]; }));
    if ((threadIdx.x & 63) == 0) p.col_sum[2 * c + q] = v;
}

hipError_t launch_col_sums(const Plan& p, const int* col_seg, const int* col_idx, hipStream_t st) {
    if (p.n_cols <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_col_sums, dim3((2 * p.n_cols + 3) / 4), dim3(256), 0, st, p.dev, col_seg, col_idx);
    return hipGetLastError();
}

// One wave per image: its three sums.
__global__ __launch_bounds__(256) void k_img_sums(PlanPtr pp, const int2* __restrict__ img_items) {
    PlanRef p = *pp;
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= p.n_images) return;
    const int2 it = img_items[k];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double v = butterfly(lane_sum(it.x, it.y, [&](int i) { return p.fwd_part[3LL * i + c]; }));
        if ((threadIdx.x & 63) == 0) p.img_sum[3 * k + c] = v;
    }
}

// One workgroup per sub-problem: for each of its images, every thread takes items tid, tid +
// 256, ... (all three components), then a fixed butterfly per wave and the four waves in order;
// thread 0 adds the images' chi^2 in order.  One launch instead of four (image sums, chi^2,
// check or accept): at 64 x 64 they were 1.8 us of work and 5 us of launch each.  An image costs
// the workgroup 0.65 us, so where a sub-problem has more than TAIL_IMAGES of them (io.summed) the
// image sums have a launch of their own, and one wave adds them (200 images in one sub-problem:
// a chi^2 call 215 us with the images one after another, 77 so).
__global__ __launch_bounds__(256) void k_tail(PlanPtr pp, TailIO io) {
    PlanRef p = *pp;
    __shared__ double red[4][3];
    __shared__ int acc_flag;
    const int s = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double chi = 0.0;                                    // thread 0's
    if (io.summed && wv == 0)
        chi = butterfly(lane_sum(io.chi_seg[s], io.chi_seg[s + 1], [&](int q) { return p.img_sum[3 * io.sub_img[q]]; }));
    for (int q = io.summed ? io.chi_seg[s + 1] : io.chi_seg[s]; q < io.chi_seg[s + 1]; ++q) {
        const int k = io.sub_img[q];
        const int2 it = io.img_items[k];
        double v0 = 0.0, v1 = 0.0, v2 = 0.0;
        for (int i = it.x + (int)threadIdx.x; i < it.y; i += 512) {
            const double* a = p.fwd_part + 3LL * i;
            const bool two = i + 256 < it.y;
            const double a0 = a[0], a1 = a[1], a2 = a[2];
            const double b0 = two ? a[768] : 0.0, b1 = two ? a[769] : 0.0, b2 = two ? a[770] : 0.0;
            v0 += a0;
            v1 += a1;
            v2 += a2;
            v0 += b0;
            v1 += b1;
            v2 += b2;
        }
        v0 = butterfly(v0);
        v1 = butterfly(v1);
        v2 = butterfly(v2);
        if (lane == 0) {
            red[wv][0] = v0;
            red[wv][1] = v1;
            red[wv][2] = v2;
        }
        __syncthreads();
        if (threadIdx.x < 3) {
            const int c = threadIdx.x;
            const double v = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
            p.img_sum[3 * k + c] = v;
            chi += v;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (io.chi2) io.chi2[s] = chi;
        if (io.kind == TAIL_CHECK && !isfinite(chi)) atomicOr(p.sticky, FLAG_NONFINITE);
        if (io.kind == TAIL_INIT) lm_init_state(p, s, chi, io.lm);
        acc_flag = io.kind == TAIL_ACCEPT ? lm_accept_state(p, s, chi, io.lm) : 0;
    }
    if (io.kind != TAIL_ACCEPT) return;
    __syncthreads();
    if (acc_flag) {
        const DSub sb = p.subs[s];
        for (int k = threadIdx.x; k < sb.n; k += 256) io.theta[sb.p0 + k] = p.theta_trial[sb.p0 + k];
    }
}

hipError_t launch_tail(const Plan& p, const TailIO& io, hipStream_t st) {
    if (io.summed) hipLaunchKernelGGL(k_img_sums, dim3((p.n_images + 3) / 4), dim3(256), 0, st, p.dev, io.img_items);
    hipLaunchKernelGGL(k_tail, dim3(p.n_sub), dim3(256), 0, st, p.dev, io);
    return hipGetLastError();
}

// One wave per column: the sum of its tile partials.
__global__ __launch_bounds__(256) void k_grad_cols(GradSum a) {
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= a.n_cols) return;
    const double v = butterfly(lane_sum(a.gcol_seg[c], a.gcol_seg[c + 1], [&](int i) { return a.grad_part[i]; }));
    if ((threadIdx.x & 63) == 0) a.src[a.col0 + c] = v;
}

// One wave per theta index.  A column costs the wave 0.75 us, so where a parameter is tied over more
// than GRAD_COLUMNS of them (a.summed) the columns have a launch of their own before it (200
// components tied, in 200 images: a gradient call 391 us before both, 104 now).
__global__ __launch_bounds__(256) void k_grad_sum(GradSum a) {
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= a.n_par) return;
    const int lane = threadIdx.x & 63;
    double acc = 0.0;
    if (a.summed) acc = lane_sum(a.gr_seg[k], a.gr_seg[k + 1], [&](int q) { return a.gr_w[q] * a.src[a.gr_idx[q]]; });
    for (int q = a.summed ? a.gr_seg[k + 1] : a.gr_seg[k]; q < a.gr_seg[k + 1]; ++q) {
        const int j = a.gr_idx[q], c = j - a.col0;
        const double w = a.gr_w[q];
        if (c >= 0 && c < a.n_cols) acc += w * lane_sum(a.gcol_seg[c], a.gcol_seg[c + 1], [&](int i) { return a.grad_part[i]; });
        else if (lane == 0) acc += w * a.src[j];
    }
    acc = butterfly(acc);
    if (lane == 0) a.out[k] = acc;
}

hipError_t launch_grad_sum(const GradSum& a, hipStream_t st) {
    if (a.n_par <= 0) return hipSuccess;
    if (a.summed && a.n_cols > 0) hipLaunchKernelGGL(k_grad_cols, dim3((a.n_cols + 3) / 4), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_grad_sum, dim3((a.n_par + 3) / 4), dim3(256), 0, st, a);
    return hipGetLastError();
}

// J^T W J assembly: every upper entry (sub, a <= b) sums its sources in list order and
// is written to both (a, b) and (b, a) of its sub-problem's row-major block.  The blocks after
// the entries' take one theta index each: J^T W r (one wave, lanes strided, fixed butterfly).
// Sub-problems that keep their Jacobian are skipped when lm is given.
constexpr int ASM_B = 8;
__global__ __launch_bounds__(64) void k_assemble(AsmA a, int ent_blocks) {
    if ((int)blockIdx.x >= ent_blocks) {
        const int k = (int)blockIdx.x - ent_blocks;
        if (a.lm && a.lm[a.g_sub[k]].need_jac == 0) return;
        const double v = butterfly(lane_sum(a.g_seg[k], a.g_seg[k + 1], [&](int i) { return a.g_w[i] * a.src[a.g_idx[i]]; }));
        if (threadIdx.x == 0) a.g[k] = v;
        return;
    }
    const long long e = (long long)blockIdx.x * 64 + threadIdx.x;
    if (e >= a.n_ent) return;
    const int s = a.ent_sub[e];
    if (a.lm && a.lm[s].need_jac == 0) return;
    // the sources' loads in batches of ASM_B, added in list order (one at a time, an entry with
    // 36 sources took 36 round trips to memory)
    double acc = 0.0;
    const long long k1 = a.ent_off[e + 1];
    for (long long k = a.ent_off[e]; k < k1; k += ASM_B) {
        long long idx[ASM_B];
        double v[ASM_B];
#pragma unroll
        for (int q = 0; q < ASM_B; ++q) idx[q] = a.ent_src[k + q < k1 ? k + q : k1 - 1];
#pragma unroll
        for (int q = 0; q < ASM_B; ++q) v[q] = a.src[idx[q]];
#pragma unroll
        for (int q = 0; q < ASM_B; ++q) acc += k + q < k1 ? v[q] : 0.0;
    }
    const DSub sb = a.subs[s];
    const int r = a.ent_row[e], c = a.ent_col[e];
    a.out[sb.a_off + (long long)r * sb.n + c] = acc;
    a.out[sb.a_off + (long long)c * sb.n + r] = acc;
}

hipError_t launch_assemble(const AsmA& a, hipStream_t st) {
    const long long eb = (a.n_ent + 63) / 64;
    if (eb + a.n_par <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_assemble, dim3((unsigned)(eb + a.n_par)), dim3(64), 0, st, a, (int)eb);
    return hipGetLastError();
}

// Dense Jacobian for callers that want it: J[k * ldJ + i] = sum of the stored blocks of
// the columns tied to theta index k (in column order) + 1 on the pixels of images whose
// sky is theta index k.
__global__ void k_jscatter(PlanPtr pp, const int* __restrict__ par_off, const int* __restrict__ par_cols,
                           const int* __restrict__ par_sky_off, const int* __restrict__ par_sky,
                           float* __restrict__ Jd, long long ldJ) {
    PlanRef p = *pp;
    const int k = blockIdx.y;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.n_pix) return;
    // image of pixel i (binary search on pix_off)
    int lo = 0, hi = p.n_images - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (p.images[mid].pix_off <= i) lo = mid; else hi = mid - 1;
    }
    const DImage& im = p.images[lo];
    const long long local = i - im.pix_off;
    const int y = (int)(local / im.Wc), x = (int)(local - (long long)y * im.Wc);
    float v = 0.f;
    for (int q = par_off[k]; q < par_off[k + 1]; ++q) {
        const DCol cl = p.cols[par_cols[q]];
        const DGroup& g = p.groups[cl.group];
        if (g.image != lo) continue;
        if (y < g.oy0 || y >= g.oy0 + g.oh || x < g.ox0 || x >= g.ox0 + g.ow) continue;
        const int ci = par_cols[q] - g.col_begin;
        v += p.J[g.j_off + (long long)ci * g.oh * g.ow + (long long)(y - g.oy0) * g.ow + (x - g.ox0)];
    }
    for (int q = par_sky_off[k]; q < par_sky_off[k + 1]; ++q)
        if (par_sky[q] == lo) v += 1.f;
    Jd[(long long)k * ldJ + i] = v;
}

hipError_t launch_jscatter(const Plan& p, const int* par_off, const int* par_cols,
                           const int* par_sky_off, const int* par_sky, float* Jd, long long ldJ,
                           hipStream_t st) {
    if (p.n_par == 0 || p.n_pix == 0) return hipSuccess;
    dim3 grid((unsigned)((p.n_pix + 255) / 256), p.n_par);
    hipLaunchKernelGGL(k_jscatter, grid, dim3(256), 0, st, p.dev, par_off, par_cols, par_sky_off,
                       par_sky, Jd, ldJ);
    return hipGetLastError();
}

__global__ void k_fill_d(double* x, long long n, double v) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        x[i] = v;
}

__global__ void k_fill_f(float* x, long long n, float v) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        x[i] = v;
}

hipError_t launch_fill_f(float* x, long long n, float v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    long long b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    hipLaunchKernelGGL(k_fill_f, dim3((unsigned)b), dim3(256), 0, st, x, n, v);
    return hipGetLastError();
}

hipError_t launch_fill(double* x, long long n, double v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    long long b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    hipLaunchKernelGGL(k_fill_d, dim3((unsigned)b), dim3(256), 0, st, x, n, v);
    return hipGetLastError();
}

}  // namespace apx
