// chol.hip -- Cholesky factorization A = L L^T of a symmetric positive
// definite matrix, the third one-sided factorization the paper's
// introduction and conclusion carry the approach over to.
//
// Blocked right-looking Cholesky.  Block columns of kOuter = 256 columns;
// inside one, panels of kPanel = 64 columns:
//
//   chol_diagonal  a 64 x 64 diagonal block in 16-column panels: a panel's
//                  steps on one wave (lane = row, the panel's entries in
//                  registers), its update of the later columns as matrix-core
//                  tiles by four waves.  The first block has a launch of its
//                  own; every later one is tile (0, 0) of the update before it,
//                  whose workgroup factors it while the other tiles run;
//   k_chol_solve   the rows below it, l_i = a_i L11^{-T}, 16 rows a wave;
//   k_chol_update  C -= W W^T on the lower triangle of a trailing block:
//                  with W the panel inside its block column (K = 64, the
//                  columns of the rest of the block column), then with W
//                  the whole block column (K = 256, the trailing matrix).
//                  FP64 matrix-core tiles over 64 x 64 output tiles of
//                  the lower triangle, operands staged through LDS in
//                  16-column chunks (double-buffered).
//
// The trailing matrix is read and written once per 256-column block
// column: 2 x 8 bytes of HBM traffic per 2 x 256 flops, which keeps the
// update on the matrix cores' side of the roofline (the
// communication-avoiding blocking of the sequential Cholesky algorithms the
// paper cites); the operands, a 256-column block of L, are re-read from
// the caches by every tile.
//
// A failed pivot (<= 0 or NaN) writes j + 1 to the info word; every later
// kernel reads the word first and returns at once.  An update whose own tile
// (0, 0) fails is not later: its other tiles may read the word before or after
// it is written, wave by wave, and finish the update either way.
#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

namespace {

constexpr int kPanel = 64;
constexpr int kOuter = 256;

// 1 / sqrt(d) for a positive normal d: the hardware estimate and two
// Newton steps r <- r (3/2 - d r^2 / 2), each squaring the relative error.
__device__ __forceinline__ double rsqrt_f64(double d) {
    double r = __builtin_amdgcn_rsq(d);
    const double hd = 0.5 * d;
    r = r * fma(-hd, r * r, 1.5);
    r = r * fma(-hd, r * r, 1.5);
    return r;
}

constexpr int kDiagLd = 65;   // row stride of a diagonal block in LDS

// Step K of panel p of a diagonal block on one wave: lane = row, its entries
// of columns 16 p .. 16 p + 15 in m; the panel's own rows 16 p + lane % 16 once
// more in dg, on every 16-lane row, so that their entries of column K of L are
// DPP operands of the updates.  Column K is left in m[K].  Entries above the
// diagonal hold values that nothing reads.  fail: the first column whose pivot
// is not positive (the steps after it go on with what is there).
template <int K>
struct DiagStep {
    __device__ __forceinline__ static void run(double (&m)[16], double (&dg)[16], int p, int &fail) {
        const double d = row_bcast<K>(dg[K]);
        fail = (fail < 0 && !(d > 0.0)) ? 16 * p + K : fail;
        const double rinv = rsqrt_f64(d);
        const double v = m[K] * rinv, vd = dg[K] * rinv;
        m[K] = v;
        row_terms<K + 1>(dg, -vd, vd);
        row_terms<K + 1>(m, -vd, v);
        if constexpr (K + 1 < 16) DiagStep<K + 1>::run(m, dg, p, fail);
    }
};

// Cholesky factor of the 64 x 64 block in S (its lower triangle; rows past
// the block's order hold the identity) by four waves, in place.  Returns the
// first column whose pivot is not positive, or -1, on wave 0.  What bounds
// it: the chain of 64 steps (pivot broadcast, reciprocal square root, the
// panel's update), about 200 cycles each; 300 with the column's entries read
// lane by lane into scalars.
__device__ __forceinline__ int chol_diagonal(double *S) {
    const int w = wave_index<4>(), lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
    int fail = -1;
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        if (w == 0) {
            double m[16], dg[16];
            double *row = S + lane * kDiagLd + 16 * p, *own = S + (16 * p + l16) * kDiagLd + 16 * p;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                m[j] = row[j];
                dg[j] = own[j];
            }
            DiagStep<0>::run(m, dg, p, fail);
#pragma unroll
            for (int j = 0; j < 16; ++j) row[j] = m[j];
        }
        __syncthreads();
        // tiles (a, s), p < s <= a, dealt to the waves
        int e = 0;
        for (int s = p + 1; s < 4; ++s)
            for (int a = s; a < 4; ++a, ++e) {
                if ((e & 3) != w) continue;
                d4 c;
#pragma unroll
                for (int r = 0; r < 4; ++r) c[r] = S[(16 * a + 4 * r + l4) * kDiagLd + 16 * s + l16];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    c = mfma_f64(-S[(16 * a + l16) * kDiagLd + 16 * p + 4 * u + l4],
                                 S[(16 * s + l16) * kDiagLd + 16 * p + 4 * u + l4], c);
#pragma unroll
                for (int r = 0; r < 4; ++r) S[(16 * a + 4 * r + l4) * kDiagLd + 16 * s + l16] = c[r];
            }
        __syncthreads();
    }
    return fail;
}

// The factored block's lower triangle to A, or the failed column to dinfo.
__device__ __forceinline__ void chol_diagonal_out(const double *S, double *__restrict__ A, int64_t lda, int64_t s,
                                                  int sb, int fail, int *flag, int32_t *__restrict__ dinfo) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (t == 0) *flag = fail;
    __syncthreads();
    if (*flag >= 0) {
        if (t == 0) *dinfo = (int32_t)(s + *flag + 1);
        return;
    }
    double *Ad = A + s + s * lda;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int c = w + 4 * u;
        if (c <= lane && lane < sb) Ad[lane + c * lda] = S[lane * kDiagLd + c];
    }
}

__global__ __launch_bounds__(64) void k_chol_info_clear(int32_t *dinfo) {
    if (threadIdx.x == 0) *dinfo = 0;
}

__global__ __launch_bounds__(256) void k_chol_diag(double *__restrict__ A, int64_t lda, int sb,
                                                   int32_t *__restrict__ dinfo) {
    __shared__ double S[kPanel * kDiagLd];
    __shared__ int flag;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int c = w + 4 * u;
        const double v = A[(c <= lane && lane < sb) ? lane + c * lda : 0];
        S[lane * kDiagLd + c] = lane < sb ? (c <= lane ? v : 0.0) : (c == lane ? 1.0 : 0.0);
    }
    __syncthreads();
    const int fail = chol_diagonal(S);
    chol_diagonal_out(S, A, lda, 0, sb, fail, &flag, dinfo);
}

// Rows s + 64 + 16 blockIdx.x + 0 .. 15 of panel s .. s + 63 against its
// factored diagonal block, on one wave (solve_rows16).  What bounds it: latency -- the
// loads, then 4 x 136 multiply-adds and 24 matrix-core tiles in a chain (about
// 5 thousand cycles); 16 rows a wave give 8,192 rows two waves per unit.
// Measured: 9.4 us a panel of 8,192 rows; 16.4 us with 64 rows a wave, all
// 2,016 multiply-adds on one lane, and 46 us for the diagonal block in every
// workgroup and the solve in one kernel.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_chol_solve(double *__restrict__ A, int64_t lda, int64_t n, int64_t s, const int32_t *__restrict__ dinfo) {
    __shared__ double X[16][17];   // [column][row]
    if (*(const volatile int32_t *)dinfo != 0) return;
    const int lane = threadIdx.x, l16 = lane & 15, l4 = lane >> 4;
    const double *__restrict__ Ld = A + s + s * lda;
    const int64_t r = s + kPanel + (int64_t)blockIdx.x * 16 + l16;
    double *__restrict__ Ar = A + (r < n ? r : n - 1) + s * lda;
    d4 c[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) c[t][q] = Ar[(16 * t + 4 * q + l4) * lda];
    double nl[4][16], dg[4], lo[4][4][4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        dg[p] = Ld[(16 * p + l16) * (lda + 1)];
#pragma unroll
        for (int k = 0; k < 16; ++k) nl[p][k] = Ld[16 * p + l16 + (16 * p + (k < l16 ? k : l16)) * lda];
#pragma unroll
        for (int t = p + 1; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) lo[p][t][q] = Ld[16 * t + l16 + (16 * p + 4 * q + l4) * lda];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) dg[p] = 1.0 / dg[p];
    solve_rows16(
        c, nl, lo, X, [&](double v, int p, int K) { return v * wave_bcast(dg[p], K); },
        [&](int col, double x) {
            if (r < n) Ar[col * lda] = x;
        });
}

// C(i, c) -= sum_{k < 16 nch} A(i, kc + k) A(c, kc + k) for t0 <= c < cend,
// c <= i < n: the lower triangle of a trailing block, by 64 x 64 tiles
// (bi, bc), bc <= bi, numbered column after column.  Four waves in a 2 x 2
// grid of 32 x 32 sub-tiles.  Tile (0, 0) is the next panel's diagonal block:
// its workgroup goes on to factor it.
// A 16-column chunk of both operands sits in LDS, two columns side by side (a
// 16-byte read feeds two products), the next chunk's loads in flight; rows
// past the end repeat the last row and nothing in the loop is conditional, so
// that the accumulators stay where the matrix cores write them.  The product
// is formed transposed: a store covers 16 rows of a column.  Measured on the
// trailing updates of 8,192 columns: 4.64 -> 3.63 ms (a branch around the
// products had moved all accumulators to other registers and back in each
// chunk, and each entry of C was loaded and waited for in front of its store).
__global__ __launch_bounds__(256, 4) void k_chol_update(double *__restrict__ A, int64_t lda, int64_t n, int64_t t0,
                                                        int64_t cend, int64_t kc, int nch, int64_t Tr, int64_t Tc,
                                                        int32_t *__restrict__ dinfo) {
    // a pivot before column t0 failed (tile (0, 0) of this launch writes t0 + 1
    // or more, which must not part a workgroup's waves)
    const int32_t failed = *(const volatile int32_t *)dinfo;
    if (failed != 0 && failed <= t0) return;
    __shared__ __attribute__((aligned(16))) double smem[kPanel * kDiagLd];   // operands, then the diagonal block
    __shared__ int flag;
    double2(*As)[8][kPanel] = reinterpret_cast<double2(*)[8][kPanel]>(smem);   // [buffer][columns 2 q, 2 q + 1][row]
    double2(*Bs)[8][kPanel] = As + 2;
    static_assert(4 * 16 * kPanel <= kPanel * kDiagLd, "both operands, double-buffered");

    // tile id -> (bi, bc): column bc starts at bc Tr - bc (bc - 1) / 2
    const int64_t id = blockIdx.x;
    int64_t lo = 0, hi = Tc - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (mid * Tr - mid * (mid - 1) / 2 <= id) lo = mid;
        else hi = mid - 1;
    }
    const int64_t bc = lo;
    const int64_t bi = bc + (id - (bc * Tr - bc * (bc - 1) / 2));
    const int64_t i0 = t0 + bi * kPanel, c0 = t0 + bc * kPanel;

    const int w = wave_index<4>(), lane = threadIdx.x & 63;
    const int wi = w >> 1, wj = w & 1;

    // wave w loads columns 4 w .. 4 w + 3 of a chunk, lane = row
    const double *Aa = A + (i0 + lane < n ? i0 + lane : n - 1) + (kc + 4 * w) * lda;
    const double *Ab = A + (c0 + lane < n ? c0 + lane : n - 1) + (kc + 4 * w) * lda;
    double ra[4], rb[4];
    auto load = [&] {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            ra[q] = Aa[q * lda];
            rb[q] = Ab[q * lda];
        }
        Aa += 16 * lda;
        Ab += 16 * lda;
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
            As[buf][2 * w + q / 2][lane] = double2{ra[q], ra[q + 1]};
            Bs[buf][2 * w + q / 2][lane] = double2{rb[q], rb[q + 1]};
        }
    };

    load();
    // this lane's entries of C: row crow of sub-tile I, columns ccol + 4 r of J
    d4 acc[2][2];
    auto crow = [&](int I) { return i0 + 32 * wi + 16 * I + d_col(lane); };
    auto ccol = [&](int J, int r) { return c0 + 32 * wj + 16 * J + d_row(r, lane); };
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J) acc[I][J] = d4_zero();
    stash(0);
    __syncthreads();
    const int ri = 32 * wi + (lane & 15), rj = 32 * wj + (lane & 15), kq = lane >> 4;
#pragma unroll 1
    for (int ch = 0; ch < nch; ++ch) {
        const int buf = ch & 1;
        if (ch + 1 < nch) load();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            double2 a[2], b[2];
#pragma unroll
            for (int I = 0; I < 2; ++I) a[I] = As[buf][4 * ks + kq][ri + 16 * I];
#pragma unroll
            for (int J = 0; J < 2; ++J) b[J] = Bs[buf][4 * ks + kq][rj + 16 * J];
#pragma unroll
            for (int I = 0; I < 2; ++I)
#pragma unroll
                for (int J = 0; J < 2; ++J) acc[I][J] = mfma_f64(b[J].x, a[I].x, acc[I][J]);
#pragma unroll
            for (int I = 0; I < 2; ++I)
#pragma unroll
                for (int J = 0; J < 2; ++J) acc[I][J] = mfma_f64(b[J].y, a[I].y, acc[I][J]);
        }
        if (ch + 1 < nch) stash(buf ^ 1);
        __syncthreads();
    }
    // C in one batch of loads, the sum subtracted from it
    d4 cc[2][2];
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // above the diagonal and past the end: an entry of the triangle, not stored
                const int64_t row = crow(I) < n ? crow(I) : n - 1, c = ccol(J, r), col = c < row ? c : row;
                cc[I][J][r] = A[row + col * lda];
            }
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J) acc[I][J] = cc[I][J] - acc[I][J];
    if (id == 0) {
        double *S = smem;
        const int sb = (int)(cend - t0 < kPanel ? cend - t0 : kPanel);
#pragma unroll
        for (int I = 0; I < 2; ++I)
#pragma unroll
            for (int J = 0; J < 2; ++J)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = (int)(crow(I) - t0), col = (int)(ccol(J, r) - t0);
                    S[row * kDiagLd + col] = (row < sb && col <= row) ? acc[I][J][r] : (row == col ? 1.0 : 0.0);
                }
        __syncthreads();
        const int fail = chol_diagonal(S);
        chol_diagonal_out(S, A, lda, t0, sb, fail, &flag, dinfo);
        return;
    }
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t row = crow(I), col = ccol(J, r);
                if (row < n && col < cend && row >= col) A[row + col * lda] = acc[I][J][r];
            }
}

// K: a multiple of 16 (whole panels).
hipError_t update(double *A, int64_t lda, int64_t n, int64_t t0, int64_t cend, int64_t kc, int K,
                  int32_t *dinfo, const char *tag, hipStream_t st) {
    const int64_t Tr = (n - t0 + kPanel - 1) / kPanel, Tc = (cend - t0 + kPanel - 1) / kPanel;
    const int64_t tiles = Tc * Tr - Tc * (Tc - 1) / 2;
    if (tiles <= 0) return hipSuccess;
    if (tiles > INT32_MAX) return hipErrorInvalidValue;
    ProfScope ps(tag, st);
    hipLaunchKernelGGL(k_chol_update, dim3((unsigned)tiles), dim3(256), 0, st, A, lda, n, t0, cend, kc, K / 16,
                       Tr, Tc, dinfo);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_cholesky(int64_t n, double *A, int64_t lda, int32_t *dinfo, hipStream_t st) {
    hipLaunchKernelGGL(k_chol_info_clear, dim3(1), dim3(64), 0, st, dinfo);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (n == 0) return hipSuccess;
    {
        ProfScope ps("chol_diag", st);
        hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(256), 0, st, A, lda, (int)(n < kPanel ? n : kPanel), dinfo);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (int64_t j = 0; j < n; j += kOuter) {
        const int64_t jend = j + kOuter < n ? j + kOuter : n;
        for (int64_t s = j; s < jend; s += kPanel) {
            const int sb = (int)(jend - s < kPanel ? jend - s : kPanel);
            const int64_t below = n - s - sb;   // none unless sb = 64
            if (below > 0) {
                ProfScope ps("chol_solve", st);
                hipLaunchKernelGGL(k_chol_solve, dim3((unsigned)((below + 15) / 16)), dim3(64), 0, st, A, lda, n, s,
                                   dinfo);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
            if (s + sb < jend) {
                e = update(A, lda, n, s + sb, jend, s, sb, dinfo, "chol_update", st);
                if (e != hipSuccess) return e;
            }
        }
        if (jend < n) {
            // 64 x 64 tiles: four resident workgroups per compute unit hide
            // the operand loads better than 128 x 128 tiles' reuse pays
            // (8192 x 8192: 4.8 against 6.4 ms of trailing updates)
            e = update(A, lda, n, jend, n, j, (int)(jend - j), dinfo, "chol_syrk", st);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace tsqr
