// panel_qr.h -- blocked Householder QR of a register-resident block of rows,
// shared by the leaf (factor.hip) and tree (tree.hip) kernels.
//
// A workgroup of W waves holds 16 W NT rows x 16 NS columns in registers:
// lane = 16 rg + cg holds column 16 t + cg of slot t, and of tile a (rows
// 16 tau .. 16 tau + 15 of the block, tau = W a + w) the rows
//     8 (r / 2) + 2 rg + r % 2,  r = 0..3,
// so that registers (0, 1) and (2, 3) are row pairs (16-byte accesses, four
// lanes on 64 consecutive bytes of a column) and a tile is at once an FP64
// matrix-core operand and result: register i of slot t holds A[m = cg][k =
// rg] or B[k = rg][n = cg] of four rows, and D[4 r + rg][cg] of a tile.
//
// The columns go in panels of 16 (one slot):
//   * 16 column steps touch only the panel's slot.  The step's column is
//     broadcast inside every 16-lane row by one DPP move per row of the tile
//     (no LDS, no shuffle), the dots are summed over the four lane rows by one
//     4x4x4 matrix product with ones and over the waves through LDS behind one
//     barrier;
//   * the panel's 16 x 16 T grows by a column per step (rows on lanes) while
//     the step waits for its barrier;
//   * the other slots get the panel as one compact-WY update (Sec. 2.2,
//     H_1..H_16 = I - V T V^T) on the FP64 matrix cores: W = V^T C straight
//     from the registers, M = T^T (R rows + W), R rows -= M, C -= V M with V
//     read back from LDS as row operands.
// What bounds it: the chain of 64 column steps.  A step costs ~2,800 cycles
// when it works on all 64 columns with the column passed through LDS; on the
// panel's slot alone its chain is the dot, two lane exchanges, one barrier,
// the Householder scalars and the update.
//
// Panels rotate through slot 0 (slot s holds columns 16 ((s + p) mod NS) at
// panel p), so one copy of the 16 unrolled steps serves every panel and the
// kernel stays inside the instruction cache.
#pragma once

#include <type_traits>

#include "common.h"
#include "mfma.h"

namespace tsqr {

// v of lane Q of the lane's 16-lane row.
template <int Q>
__device__ __forceinline__ double row_bcast(double v) {
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + Q, 0xf, 0xf, true);
}

// The wave's index in its workgroup (a scalar).
template <int W>
__device__ __forceinline__ int wave_index() {
    if constexpr (W == 1) return 0;
    else return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Row of a 16-row tile that register r of a lane in lane row rg holds.
__device__ __forceinline__ int tile_row(int r, int rg) { return 8 * (r >> 1) + 2 * rg + (r & 1); }

// LDS of the panel steps and updates (W waves, NS slots, NT tiles a wave).
template <int W, int NS, int NT>
struct PanelSmem {
    static constexpr int kLd = 16 * NS + 1;        // row stride of R and T (odd)
    static constexpr int kVtLd = 16 * NT + 4;      // column stride of the row operands
    alignas(32) double R[16 * NS * kLd];           // running triangle, row-major
    double T[16 * NS * kLd];                       // the block's T
    alignas(32) double red[2][16 * W];             // per-wave dots of the panel's columns
    double redq[2][16];                            // pivot-row values (first block)
    alignas(32) double vt[NS > 1 ? W * 16 * kVtLd : 1];   // V of the panel by columns, a region per wave
    alignas(32) double part[(NS > 1 && W > 1) ? (NS - 1) * W * 256 : 1];   // per-wave V^T C
    double P[NS > 1 ? 16 * NS * 16 : 1];           // scratch of the block's T
};

// The step's dots over four tiles, s_r += x c with x = the register of lane Q
// of the lane's 16-lane row, as DPP operands of the FMAs (the broadcast costs
// no instruction and no register).  A DPP operand must have been written two
// wait states before: the s_nop covers the compiler's last instruction ahead
// of the block.
template <int Q>
__device__ __forceinline__ void tile_dots(double (&s)[4], const d4 &c, const d4 &d, const d4 &e, const d4 &f) {
#define TSQR_DOT(acc, x) "v_fmac_f64_dpp %" #acc ", %" #x ", %" #x " row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
    asm("s_nop 1\n\t"
        TSQR_DOT(0, 4) TSQR_DOT(1, 5) TSQR_DOT(2, 6) TSQR_DOT(3, 7)
        TSQR_DOT(0, 8) TSQR_DOT(1, 9) TSQR_DOT(2, 10) TSQR_DOT(3, 11)
        TSQR_DOT(0, 12) TSQR_DOT(1, 13) TSQR_DOT(2, 14) TSQR_DOT(3, 15)
        TSQR_DOT(0, 16) TSQR_DOT(1, 17) TSQR_DOT(2, 18) TSQR_DOT(3, 19)
        : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3])
        : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(d[0]), "v"(d[1]), "v"(d[2]), "v"(d[3]),
          "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "n"(Q));
#undef TSQR_DOT
}
// c_r += x_r f for two tiles (f = 0 in lane Q, so the broadcast column keeps
// its values).
template <int Q>
__device__ __forceinline__ void tile_axpy(d4 &c, d4 &d, double f) {
#define TSQR_AXPY(x) "v_fmac_f64_dpp %" #x ", %" #x ", %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
    double c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3], d0 = d[0], d1 = d[1], d2 = d[2], d3 = d[3];
    asm("s_nop 1\n\t"
        TSQR_AXPY(0) TSQR_AXPY(1) TSQR_AXPY(2) TSQR_AXPY(3) TSQR_AXPY(4) TSQR_AXPY(5) TSQR_AXPY(6) TSQR_AXPY(7)
        : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3), "+v"(d0), "+v"(d1), "+v"(d2), "+v"(d3)
        : "v"(f), "n"(Q));
#undef TSQR_AXPY
    c = d4{c0, c1, c2, c3};
    d = d4{d0, d1, d2, d3};
}

// The same for one tile.
template <int Q>
__device__ __forceinline__ void tile_dots(double (&s)[4], const d4 &c) {
#define TSQR_DOT(acc, x) "v_fmac_f64_dpp %" #acc ", %" #x ", %" #x " row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
    asm("s_nop 1\n\t" TSQR_DOT(0, 4) TSQR_DOT(1, 5) TSQR_DOT(2, 6) TSQR_DOT(3, 7)
        : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3])
        : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "n"(Q));
#undef TSQR_DOT
}
template <int Q>
__device__ __forceinline__ void tile_axpy(d4 &c, double f) {
#define TSQR_AXPY(x) "v_fmac_f64_dpp %" #x ", %" #x ", %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
    double c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
    asm("s_nop 1\n\t" TSQR_AXPY(0) TSQR_AXPY(1) TSQR_AXPY(2) TSQR_AXPY(3)
        : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3)
        : "v"(f), "n"(Q));
#undef TSQR_AXPY
    c = d4{c0, c1, c2, c3};
}

// Sum over the four lane rows (lanes cg, cg + 16, cg + 32, cg + 48), the
// same in all of them: a 4x4x4 FP64 matrix product with a left factor of
// ones sums its k index, which is the lane row (about half the latency of
// two permlane exchanges).
__device__ __forceinline__ double lane_rows_sum(double v) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, v, 0.0, 0, 0, 0);
}

// The wait states between a matrix-core result and the first read by the asm
// blocks above, which the compiler's hazard checks do not look into (18 for
// a 16-pass FP64 instruction).
__device__ __forceinline__ void settle(d4 &c) {
    double c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
    asm volatile("s_nop 15\n\ts_nop 3" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
    c[0] = c0;
    c[1] = c1;
    c[2] = c2;
    c[3] = c3;
}

// Householder scalars for x = [alpha; x2], ||x2||^2 = sig2 (Sec. 2.2, H = I -
// tau v v^T, LAPACK's sign convention, sgn(0) = +1): d = alpha - beta,
// s = 1 / d (v = [1; s x2]), g = tau s = sgn / |beta|, tau = g d; g = tau = 0
// if sig2 == 0 (H = I, R's entry stays alpha).  1 / |beta| is v_rsq_f64 and
// one third-order step, 1 / d v_rcp_f64 of the unrefined d and one
// third-order step on the refined one, so the two short chains overlap.
// kTiny keeps x > 0 without a branch: the smallest denormal, at most one unit in
// the last place of any normal x (norms from 2^-511 on, where ||x2||^2 leaves the
// normal range; with x = kTiny every product below is finite).
__device__ __forceinline__ void panel_scalars(double alpha, double sig2, double &beta, double &tau, double &s,
                                              double &g, double &d) {
    constexpr double kTiny = 0x1p-1074;
    const double x = fma(alpha, alpha, sig2) + kTiny;
    const double sgn = (alpha < 0.0) ? -1.0 : 1.0;
    const double r0 = __builtin_amdgcn_rsq(x);
    const double s0 = __builtin_amdgcn_rcp(fma(sgn, x * r0, alpha));
    // r = r0 (1 + e / 2 + 3 e^2 / 8), e = 1 - x r0^2
    const double e = fma(-x * r0, r0, 1.0);
    const double r = fma(r0 * e, fma(0.375, e, 0.5), r0);
    const double ab = x * r;           // |beta|
    d = fma(sgn, ab, alpha);
    const double h = fma(-d, s0, 1.0);
    s = fma(s0, fma(h, h, h), s0);
    g = (sig2 == 0.0) ? 0.0 : sgn * r;
    tau = g * d;
    beta = -sgn * ab;
}

// What a wave carries through a panel's steps.
struct PanelRegs {
    double trow[16];   // row cg of the panel's T
    double scale;      // s of this lane's column once it is a reflector
    double rrow[4];    // R rows 16 p + 4 u + rg, this lane's column
    double gq, tau;    // last step's Gram entry of this lane's column, and its tau
};

__device__ __forceinline__ void panel_begin(PanelRegs &pr) {
    pr.scale = 1.0;
    pr.gq = 0.0;
    pr.tau = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) pr.trow[q] = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) pr.rrow[u] = 0.0;
}

// Column J of the panel's T (rows on lanes) from the Gram entries of step J:
// T[0:J, J] = -tau_J T[0:J, 0:J] G[0:J, J], T_JJ = tau_J.  Lane K's Gram
// entry is a DPP operand, as in tile_dots; the first block's output stands
// for the entries in the others, so the wait states are behind all of them.
template <int K>
__device__ __forceinline__ void t_term(double &acc, double g, double t) {
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(g), "v"(t), "n"(K));
}
// u[j] += g(lane j of the 16-lane row) t, j = J0 .. 15.
template <int J>
struct RowTerms {
    __device__ __forceinline__ static void run(double (&u)[16], double g, double t) {
        if constexpr (J < 16) {
            t_term<J>(u[J], g, t);
            RowTerms<J + 1>::run(u, g, t);
        }
    }
};
template <int J0>
__device__ __forceinline__ void row_terms(double (&u)[16], double g, double t) {
    asm("s_nop 1" : "+v"(g));
    RowTerms<J0>::run(u, g, t);
}
// x L^T = a on 16 columns of one row (lane = row, u[j] its columns): x_K =
// scale(u[K], K), then u[j] -= x_K L(j, K), j > K, with row j of -L in lane j of
// every 16-lane row (column K: nl[K]).
template <int K, typename F>
__device__ __forceinline__ void lower_solve(double (&u)[16], const double (&nl)[16], F scale) {
    u[K] = scale(u[K], K);
    if constexpr (K < 15) {
        row_terms<K + 1>(u, nl[K], u[K]);
        lower_solve<K + 1>(u, nl, scale);
    }
}

// x L^T = a for 16 rows (lane % 16) and 64 columns on one wave, right-looking
// over four 16-column tiles.  c[t]: tile t as a transposed matrix-core
// accumulator (column 16 t + 4 q + lane / 16 in register q); nl[p][k]: L(16 p +
// lane % 16, 16 p + k), used for k < lane % 16; lo[p][t][q]: L(16 t + lane % 16,
// 16 p + 4 q + lane / 16), t > p.  A tile's turn: through LDS, so that every
// 16-lane row holds whole rows of it, solved, handed to out(column, x) and
// applied to the tiles after it.  scale(v, p, K): the division by L's diagonal
// entry 16 p + K.
template <typename S, typename F>
__device__ __forceinline__ void solve_rows16(d4 (&c)[4], double (&nl)[4][16], const double (&lo)[4][4][4],
                                             double (&X)[16][17], S scale, F out) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int q = 0; q < 4; ++q) X[4 * q + l4][l16] = c[p][q];
        __syncthreads();
        double u[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) u[k] = X[k][l16];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) nl[p][k] = k < l16 ? -nl[p][k] : 0.0;
        lower_solve<0>(u, nl[p], [&](double v, int K) { return scale(v, p, K); });
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double x = l4 & 2 ? (l4 & 1 ? u[4 * q + 3] : u[4 * q + 2]) : (l4 & 1 ? u[4 * q + 1] : u[4 * q]);
            out(16 * p + 4 * q + l4, x);
#pragma unroll
            for (int t = p + 1; t < 4; ++t) c[t] = mfma_f64(-lo[p][t][q], x, c[t]);
        }
    }
}

template <int J, int K>
struct TColumn {
    __device__ __forceinline__ static void run(const PanelRegs &pr, double g, double &a0, double &a1) {
        if constexpr (K < J) {
            t_term<K>(K % 2 == 0 ? a0 : a1, g, pr.trow[K]);
            TColumn<J, K + 1>::run(pr, g, a0, a1);
        }
    }
};
template <int J>
__device__ __forceinline__ void t_column(PanelRegs &pr, int cg) {
    double a0 = 0.0, a1 = 0.0, g = pr.gq;
    if constexpr (J > 0) asm("s_nop 1" : "+v"(g));
    TColumn<J, 0>::run(pr, g, a0, a1);
    pr.trow[J] = (cg < J) ? -pr.tau * (a0 + a1) : ((cg == J) ? pr.tau : 0.0);
}

// Steps Q .. 7 or Q .. 15 of panel p (column j = 16 p + Q; Rp: the panel's
// diagonal block of R, row stride ld; own_w: the wave holds the pivot rows of
// a first block).  A column past n
// is zero, and so are its scalars: such a step changes nothing.
// FIRST: plain QR of the block, whose rows 0 .. n - 1 become R (row j sits
// in tile 0 of wave p); else the structured QR of [R; block].  With x =
// column j (without the pivot row), d_k = x . c_k and e_k the pivot row's or
// R's entry of column k:
//     k > j:  w = e_k + s d_k,  c_k -= g w x,  R[j][k] = e_k - g w d,
//     k = j:  R[j][j] = beta, the column keeps x and its scale s waits,
//     k < j:  G[k][j] = y_k . y_j = s_k w.
template <int W, int NT, bool FIRST, int Q>
struct PanelStep {
    template <typename SM, typename H>
    __device__ __forceinline__ static void run(d4 (&c)[NT], PanelRegs &pr, SM &sm, const double *Rp, const int ld,
                                               const bool own_w, const int w, const int rg, const int cg, H &hook) {
        constexpr int RP = 2 * (Q / 8) + Q % 2;
        const bool own = FIRST && own_w && rg == (Q % 8) / 2;
        const double piv = c[0][RP];
        if constexpr (FIRST) c[0][RP] = own ? 0.0 : piv;
        double s4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int a = 0; a < NT; a += (NT % 4 == 0) ? 4 : 1) {
            if constexpr (NT % 4 == 0) tile_dots<Q>(s4, c[a], c[a + 1], c[a + 2], c[a + 3]);
            else tile_dots<Q>(s4, c[a]);
        }
        double dk = lane_rows_sum((s4[0] + s4[1]) + (s4[2] + s4[3]));
        // R's row j changes only in this step, behind the barrier
        double ek = 0.0;
        if constexpr (!FIRST) ek = Rp[Q * ld + cg];
        if constexpr (W > 1) {
            constexpr int par = Q & 1;
            if (rg == 0) sm.red[par][16 * w + cg] = dk;
            if constexpr (FIRST) {
                if (own) sm.redq[par][cg] = piv;
            }
            __syncthreads();
            // lane row r takes wave r's dots
            const double part = sm.red[par][16 * rg + cg];
            if constexpr (FIRST) ek = sm.redq[par][cg];
            hook(std::integral_constant<int, Q>{});
            // the last step's column of T while the reads are under way
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (Q % 8 != 0) t_column<Q - 1>(pr, cg);
            __builtin_amdgcn_sched_barrier(0);
            dk = lane_rows_sum(part);
        } else if constexpr (Q % 8 != 0) {
            t_column<Q - 1>(pr, cg);
        }
        const double sig2 = row_bcast<Q>(dk), alpha = row_bcast<Q>(ek);
        double beta, tau, s, g, d;
        panel_scalars(alpha, sig2, beta, tau, s, g, d);
        const double wv = fma(s, dk, ek);
        const double f = (cg > Q) ? -(g * wv) : 0.0;
#pragma unroll
        for (int a = 0; a < NT; a += (NT % 2 == 0) ? 2 : 1) {
            if constexpr (NT % 2 == 0) tile_axpy<Q>(c[a], c[a + 1], f);
            else tile_axpy<Q>(c[a], f);
        }
        if constexpr (FIRST) c[0][RP] = (own && cg < Q) ? piv : c[0][RP];
        {
            // row j of R: kept by the lanes of row Q mod 4 until the panel's end
            const double v = (cg == Q) ? (sig2 == 0.0 ? alpha : beta) : fma(f, d, ek);
            pr.rrow[Q / 4] = (rg == Q % 4) ? v : pr.rrow[Q / 4];
            // now, not at the panel's end with every step's scalars kept for it
            asm volatile("" : "+v"(pr.rrow[Q / 4]));
        }
        pr.gq = pr.scale * wv;
        pr.tau = tau;
        pr.scale = (cg == Q) ? s : pr.scale;
        if constexpr (Q % 8 == 7) t_column<Q>(pr, cg);
        if constexpr (Q + 1 < 16 && Q != 7)
            PanelStep<W, NT, FIRST, Q + 1>::run(c, pr, sm, Rp, ld, own_w, w, rg, cg, hook);
    }
};

// Panel p of panel_qr (below).
template <int W, int NS, int NT, bool FIRST, typename H, typename F1, typename F2>
__device__ __forceinline__ void panel_one(const int p, d4 (&c)[NS][NT], const int n, PanelSmem<W, NS, NT> &sm,
                                          const bool want_t, H hook, F1 done, F2 t_block) {
    using SM = PanelSmem<W, NS, NT>;
    constexpr int LD = SM::kLd;
    const int lane = threadIdx.x & 63, w = wave_index<W>(), rg = lane >> 4;
    const int np = (n + 15) >> 4;
    double *vt = sm.vt + (NS > 1 ? w * 16 * SM::kVtLd : 0);
    // T[w block, p] from the products P of panel p
    auto t_above = [&](int p) {
        if constexpr (NS > 1) {
            if (w < p) {
                const int cg = lane & 15;
                d4 acc = d4_zero();
#pragma unroll
                for (int u = 0; u + 1 < NS; ++u) {
                    if (w + u < p) {
#pragma unroll
                        for (int kb = 0; kb < 4; ++kb) {
                            const int k = 16 * (w + u) + 4 * kb + rg;
                            acc = mfma_f64(sm.T[(16 * w + cg) * LD + k], sm.P[k * 16 + cg], acc);
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) sm.T[(16 * w + 4 * r + rg) * LD + 16 * p + cg] = -acc[r];
            }
        }
    };
    {
        const int nq = n - 16 * p < 16 ? n - 16 * p : 16;
        int cg = lane & 15;
        asm volatile("" : "+v"(cg));   // lane masks are formed in the panel, not kept across it
        PanelRegs pr;
        panel_begin(pr);
        if constexpr (NS > 1) {
#pragma unroll
            for (int a = 0; a < NT; ++a) settle(c[0][a]);
        }
        double *Rp = sm.R + 16 * p * (LD + 1);   // the panel's diagonal block of R
        PanelStep<W, NT, FIRST, 0>::run(c[0], pr, sm, Rp, LD, w == p, w, rg, cg, hook);
        if (nq > 8) PanelStep<W, NT, FIRST, 8>::run(c[0], pr, sm, Rp, LD, w == p, w, rg, cg, hook);
        if (w == 0) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (cg >= 4 * u + rg) Rp[(4 * u + rg) * LD + cg] = pr.rrow[u];
        }
        // reflectors: v = s x, and the unit diagonal of a first block
#pragma unroll
        for (int a = 0; a < NT; ++a) c[0][a] *= pr.scale;
        if constexpr (FIRST) {
            if (w == p) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (tile_row(r, rg) == cg && cg < nq) c[0][0][r] = 1.0;
            }
        }
        double *Tp = sm.T + 16 * p * (LD + 1);   // its diagonal block of T
        if (w == 0 && rg == 0) {
#pragma unroll
            for (int q = 0; q < 16; ++q) Tp[cg * LD + q] = pr.trow[q];
        }
        done(p, c[0], pr.trow);
        if constexpr (NS > 1) {
            const int ntr = np - p;          // slots 1 .. ntr - 1: columns still to update
            if (p + 1 < np || want_t) {
                // row operands of V
#pragma unroll
                for (int a = 0; a < NT; ++a)
                    *reinterpret_cast<d4 *>(vt + cg * SM::kVtLd + 16 * a + 4 * rg) = c[0][a];
                d4 acc[NS], ev[NS];
#pragma unroll
                for (int s = 1; s < NS; ++s) {
                    acc[s] = d4_zero();
                    ev[s] = d4_zero();
                    if (!FIRST && s < ntr) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            ev[s][r] = sm.R[(16 * p + 4 * r + rg) * LD + 16 * (p + s) + cg];
                    }
                }
                // V^T C of the columns to update; V_p^T V_t of finished ones
#pragma unroll
                for (int s = 1; s < NS; ++s) {
                    if (s < ntr || (want_t && s >= NS - p)) {
#pragma unroll
                        for (int a = 0; a < NT; ++a) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) acc[s] = mfma_f64(c[0][a][r], c[s][a][r], acc[s]);
                        }
                    }
                }
                if constexpr (W > 1) {
#pragma unroll
                    for (int s = 1; s < NS; ++s)
                        *reinterpret_cast<d4 *>(sm.part + (((s - 1) * W + w) * 64 + lane) * 4) = acc[s];
                    __syncthreads();
                    if (p > 0 && want_t) t_block(p - 1);
#pragma unroll
                    for (int s = 1; s < NS; ++s) {
                        const bool gram = want_t && s >= NS - p && w == s + p - NS;
                        if (s < ntr || gram) {
                            const double *q = sm.part + ((s - 1) * W * 64 + lane) * 4;
                            acc[s] = *reinterpret_cast<const d4 *>(q);
#pragma unroll
                            for (int u = 1; u < W; ++u) acc[s] += *reinterpret_cast<const d4 *>(q + 256 * u);
                            if (gram) {
                                d4 pg = d4_zero();
#pragma unroll
                                for (int kb = 0; kb < 4; ++kb)
                                    pg = mfma_f64(acc[s][kb], Tp[(4 * kb + rg) * LD + cg], pg);
#pragma unroll
                                for (int r = 0; r < 4; ++r) sm.P[(16 * w + 4 * r + rg) * 16 + cg] = pg[r];
                            }
                        }
                    }
                }
                if (p + 1 < np) {
                    // M = T^T (R rows + W), -M kept
                    double ta[4];
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb) ta[kb] = -Tp[(4 * kb + rg) * LD + cg];
                    d4 mm[NS];
#pragma unroll
                    for (int s = 1; s < NS; ++s) {
                        if (s < ntr) {
                            const d4 wf = acc[s] + ev[s];
                            mm[s] = d4_zero();
#pragma unroll
                            for (int kb = 0; kb < 4; ++kb) mm[s] = mfma_f64(ta[kb], wf[kb], mm[s]);
                            if (!FIRST && w == (s % W)) {
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    sm.R[(16 * p + 4 * r + rg) * LD + 16 * (p + s) + cg] = ev[s][r] + mm[s][r];
                            }
                        }
                    }
                    // C -= V M
#pragma unroll
                    for (int a = 0; a < NT; ++a) {
                        double av[4];
#pragma unroll
                        for (int kb = 0; kb < 4; ++kb)
                            av[kb] = vt[(4 * kb + rg) * SM::kVtLd + 16 * a + 4 * (cg & 3) + (cg >> 2)];
#pragma unroll
                        for (int s = 1; s < NS; ++s) {
                            if (s < ntr) {
#pragma unroll
                                for (int kb = 0; kb < 4; ++kb) c[s][a] = mfma_f64(av[kb], mm[s][kb], c[s][a]);
                            }
                        }
                    }
                    if constexpr (FIRST) {
                        // the pivot rows of the other columns become R rows
                        if (w == p) {
#pragma unroll
                            for (int s = 1; s < NS; ++s) {
                                if (s < ntr) {
#pragma unroll
                                    for (int r = 0; r < 4; ++r)
                                        sm.R[(16 * p + tile_row(r, rg)) * LD + 16 * (p + s) + cg] = c[s][0][r];
                                    c[s][0] = d4_zero();
                                }
                            }
                        }
                    }
                }
            }
            // the finished panel to the last slot
            d4 t0[NT];
#pragma unroll
            for (int a = 0; a < NT; ++a) t0[a] = c[0][a];
#pragma unroll
            for (int s = 0; s + 1 < NS; ++s)
#pragma unroll
                for (int a = 0; a < NT; ++a) c[s][a] = c[s + 1][a];
#pragma unroll
            for (int a = 0; a < NT; ++a) c[NS - 1][a] = t0[a];
        }
        // R rows updated above are read by the next panel's steps, P by t_above
        if constexpr (W > 1) __syncthreads();
        if (want_t) t_above(p);
    }
}

// Householder QR of the block c (FIRST) or of [R; c] (R: sm.R).  On exit
// sm.R is the new triangle and, if want_t, sm.T the block's T.
// `hook0` runs in every step of panel 0 while the step waits for LDS, `hook`
// in every step of the later panels (slot NS - 1 then holds the panel
// before); a panel of at most 8 columns has steps 0 .. 7 only.
// `done(p, v, trow)` runs once panel p's reflector columns v (FIRST: with
// the unit diagonal of the pivot rows written out and zeros above it) and
// the rows of its T are final, and `t_block(p)` once the columns 16 p ..
// 16 p + 15 of T are in sm.T. PEEL: panel 0 has
// code of its own.
//
// T above its diagonal blocks comes from the Gram blocks G = V_t^T V_p of the
// finished panels t < p: T[0:16p, p] = -T[0:16p, 0:16p] (G[0:16p, p] T_pp),
// block row t by wave t (the summed Gram block is that wave's left operand
// as it stands; the products P_t = G_tp T_pp are exchanged through LDS over
// the barrier that ends the panel).
template <int W, int NS, int NT, bool FIRST, bool PEEL, typename H0, typename H, typename F1, typename F2>
__device__ __forceinline__ void panel_qr(d4 (&c)[NS][NT], const int n, PanelSmem<W, NS, NT> &sm, const bool want_t,
                                         H0 hook0, H hook, F1 done, F2 t_block) {
    static_assert(W == 4 && NS <= W + 1, "lane rows sum the waves; a wave per block row of T");
    const int np = (n + 15) >> 4;
    if constexpr (PEEL) panel_one<W, NS, NT, FIRST>(0, c, n, sm, want_t, hook0, done, t_block);
    if constexpr (NS > 1 || !PEEL) {
#pragma unroll 1
        for (int p = PEEL ? 1 : 0; p < np; ++p)
            panel_one<W, NS, NT, FIRST>(p, c, n, sm, want_t, hook, done, t_block);
    }
    if (want_t) {
        __syncthreads();
        t_block(np - 1);
    }
}

}  // namespace tsqr
