// calu.hip -- LU of an m x n matrix (m >= n) with tournament pivoting
// (CALU), the LU counterpart of CAQR that the paper's conclusion names
// beside TSLU.  Panels of 64 columns; panel k:
//
//   TSLU (tslu.hip) of the m - k rows below the diagonal: the tournament's
//     pivot rows, U11 and L = A U11^{-1} in the panel's row order;
//   k_calu_swaps   one wave turns the pivot rows into LAPACK-style row
//                  interchanges (interchange i swaps rows k + i and
//                  k + swp[i], swp[i] = where the i-th pivot row sits after
//                  interchanges 0..i-1) and merges the panel's info word;
//   k_calu_rowswap the interchanges on every column outside the panel, as
//                  one gather per column over the touched positions;
//   k_calu_pack    the panel's columns in the permuted row order: U on and
//                  above the diagonal block's diagonal, L below (row rel
//                  takes the L row of the original row that the interchanges
//                  brought there);
//   k_calu_trsm    U12 = L11^{-1} A12 by forward substitution (unit
//                  diagonal), 16 columns a wave in four 16-row tiles, each
//                  applied to the later ones on the matrix cores;
//   k_lu_update    A22 -= L21 U12 on the FP64 matrix cores, 64 x 64 tiles,
//                  operands staged through LDS in 16-deep chunks.
#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

namespace {

constexpr int kLuPanel = 64;

// Per-panel interchange record (int32 words): swp[0..63], then the touched
// positions (at most 128: the top b and the displaced ones), the row each
// ends up holding (its position before the panel's interchanges), and their
// count.
constexpr int kMetaSwp = 0, kMetaPos = 64, kMetaSrc = 192, kMetaCount = 320;

__global__ __launch_bounds__(64) void k_calu_clear(int32_t *dinfo) {
    if (threadIdx.x == 0) *dinfo = 0;
}

// swp[i] from the pivot rows piv (relative to row k), on one wave.  Lane t
// tracks the row at position t < b (top) and one position at or past b that
// an interchange has filled with another row (the displaced list, nd
// entries); every other position holds its own row.  Step i finds where
// piv[i] sits by a ballot over both, exchanges it with position i and
// records the row it displaces.  ipiv_out[i] = k + swp[i].  The touched
// positions and the rows they end up holding go to meta (see CaluMeta) for
// the row exchange.  dinfo <- k + pinfo on the first panel whose U has an
// exactly zero diagonal entry.
__global__ __launch_bounds__(64) void k_calu_swaps(const int64_t *__restrict__ piv, int b, int64_t k,
                                                   int32_t *__restrict__ meta, int64_t *__restrict__ ipiv_out,
                                                   const int32_t *__restrict__ pinfo, int32_t *__restrict__ dinfo) {
    int32_t *__restrict__ swp = meta + kMetaSwp;
    const int t = threadIdx.x;
    __shared__ int64_t pv[kLuPanel];
    if (t < b) pv[t] = piv[t];
    __syncthreads();
    int64_t top = t, dpos = -1, drow = -1;
    int nd = 0;
    int64_t mine = 0;   // swp[t], kept by lane t
    for (int i = 0; i < b; ++i) {
        const int64_t r = pv[i];
        const uint64_t m1 = __ballot(t >= i && t < b && top == r);
        const uint64_t m2 = __ballot(t < nd && drow == r);
        int64_t p;
        int dl = -1;
        if (m1) {
            p = __builtin_ctzll(m1);
        } else if (m2) {
            dl = __builtin_ctzll(m2);
            const int64_t dp = dpos;
            p = (int64_t)__shfl(dp, dl);
        } else {
            p = r;
        }
        const int64_t tp = top;
        const int64_t ri = __shfl(tp, i);   // the row at position i, displaced to p
        if (t == i) {
            top = r;
            mine = p;
        }
        if (p < b) {
            if (t == p && p != i) top = ri;
        } else if (dl >= 0) {
            if (t == dl) drow = ri;
        } else {
            if (t == nd) {
                dpos = p;
                drow = ri;
            }
            ++nd;
        }
    }
    if (t < b) {
        swp[t] = (int32_t)mine;
        ipiv_out[t] = k + mine;
        meta[kMetaPos + t] = t;
        meta[kMetaSrc + t] = (int32_t)top;
    }
    if (t < nd) {
        meta[kMetaPos + b + t] = (int32_t)dpos;
        meta[kMetaSrc + b + t] = (int32_t)drow;
    }
    if (t == 0) meta[kMetaCount] = b + nd;
    if (t == 0) {
        const int32_t pi = *pinfo;
        if (pi > 0 && *dinfo == 0) *dinfo = (int32_t)(k + pi);
    }
}

// Columns outside [k, k + b): the interchanges as one gather per column
// (the touched positions take the rows recorded for them; all loads of a
// column are issued before its stores).  Four columns per workgroup, one
// wave each, two touched positions per lane.
__global__ __launch_bounds__(256) void k_calu_rowswap(double *__restrict__ A, int64_t lda, int64_t n, int64_t k,
                                                      int b, const int32_t *__restrict__ meta) {
    const int lane = threadIdx.x & 63;
    int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int cnt = meta[kMetaCount];
    const bool live = c < n - b;
    if (c >= k) c += b;
    double *col = A + (live ? c : 0) * lda + k;
    const bool q0 = live && lane < cnt, q1 = live && lane + 64 < cnt;
    const int p0 = q0 ? meta[kMetaPos + lane] : 0, p1 = q1 ? meta[kMetaPos + lane + 64] : 0;
    const double v0 = q0 ? col[meta[kMetaSrc + lane]] : 0.0;
    const double v1 = q1 ? col[meta[kMetaSrc + lane + 64]] : 0.0;
    __syncthreads();
    if (q0) col[p0] = v0;
    if (q1) col[p1] = v1;
}

// Panel columns, row rel = 0 .. mr - 1 below row k: the original row o that
// the interchanges brought to rel (walk them backwards), then U11[rel][j]
// for rel < b, j >= rel, else L[o][j] (L: mr x b, ld ldl).
__global__ __launch_bounds__(256) void k_calu_pack(double *__restrict__ A, int64_t lda, int64_t mr, int64_t k,
                                                   int b, const int32_t *__restrict__ meta,
                                                   const double *__restrict__ L, int64_t ldl,
                                                   const double *__restrict__ U, int64_t ldu) {
    __shared__ int32_t s[kLuPanel];
    if (threadIdx.x < b) s[threadIdx.x] = meta[kMetaSwp + threadIdx.x];
    __syncthreads();
    const int64_t rel = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (rel >= mr) return;
    int64_t o = rel;
    for (int i = b - 1; i >= 0; --i) {
        if (o == i) o = s[i];
        else if (o == s[i]) o = i;
    }
    double *dst = A + (k + rel) + k * lda;
    double v[kLuPanel];
#pragma unroll
    for (int j = 0; j < kLuPanel; ++j)
        v[j] = (j < b) ? ((rel < b && j >= rel) ? U[rel + j * ldu] : L[o + j * ldl]) : 0.0;
#pragma unroll
    for (int j = 0; j < kLuPanel; ++j)
        if (j < b) dst[j * lda] = v[j];
}

// U12 = L11^{-1} A12 for columns k + 64 + 16 blockIdx.x + 0 .. 15 (L11: the
// unit lower triangle at k of the packed A; a panel with columns after it has
// 64), on one wave: as rows x of x L11^T = a (solve_rows16).  Measured: 4,096 x
// 4,096's 63 panels 1.65 -> 0.59 ms, against a thread per column with L11's
// columns read from LDS.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_calu_trsm(double *__restrict__ A, int64_t lda, int64_t n, int64_t k) {
    __shared__ double X[16][17];
    const int lane = threadIdx.x, l16 = lane & 15, l4 = lane >> 4;
    const double *__restrict__ Ld = A + k + k * lda;
    const int64_t c0 = k + kLuPanel + (int64_t)blockIdx.x * 16 + l16;
    double *__restrict__ col = A + k + (c0 < n ? c0 : n - 1) * lda;
    d4 c[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) c[t][q] = col[16 * t + 4 * q + l4];
    double nl[4][16], lo[4][4][4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int i = 0; i < 16; ++i) nl[p][i] = Ld[16 * p + l16 + (int64_t)(16 * p + (i < l16 ? i : l16)) * lda];
#pragma unroll
        for (int t = p + 1; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) lo[p][t][q] = Ld[16 * t + l16 + (int64_t)(16 * p + 4 * q + l4) * lda];
    }
    solve_rows16(
        c, nl, lo, X, [](double v, int, int) { return v; },
        [&](int i, double x) {
            if (c0 < n) col[i] = x;
        });
}

// A(i, c) -= sum_{kk < 64} A(i, k + kk) A(k + kk, c) for i in [r0, m),
// c in [r0, n), r0 = k + 64: 64 x 64 tiles (bi = id mod Tr, bc = id / Tr),
// four waves in a 2 x 2 grid of 32 x 32 sub-tiles, the product formed
// transposed (a store covers 16 rows of a column).  A 16-deep chunk of both
// operands sits in LDS, two depths side by side (a 16-byte read feeds two
// products), the next chunk's loads in flight; rows and columns past the end
// repeat the last one and nothing in the loop is conditional; C is read in one
// batch.  Measured: 4,096 x 4,096's 63 updates 2.63 -> 1.79 ms, against guarded
// loads with their own addresses and a wait for each entry of C.
// (Only the last panel is narrower than 64, and nothing follows it.)
__global__ __launch_bounds__(256, 4) void k_lu_update(double *__restrict__ A, int64_t lda, int64_t m, int64_t n,
                                                      int64_t k, int64_t Tr) {
    constexpr int TILE = 64, NCH = kLuPanel / 16;
    __shared__ double2 As[2][8][TILE], Bs[2][8][TILE];   // [buffer][depths 2 q, 2 q + 1][row or column]
    const int64_t r0 = k + kLuPanel;
    const int64_t bi = (int64_t)blockIdx.x % Tr, bc = (int64_t)blockIdx.x / Tr;
    const int64_t i0 = r0 + bi * TILE, c0 = r0 + bc * TILE;
    const int w = wave_index<4>(), lane = threadIdx.x & 63;
    const int wi = w >> 1, wj = w & 1;

    // A operand: row i0 + lane, depths 4 w ..; B operand: depths 2 (lane & 7)
    // .. + 1 (16 consecutive rows of U12 over 8 lanes), columns c0 + 16 w +
    // lane / 8 and 8 further on
    const double *Aa = A + (i0 + lane < m ? i0 + lane : m - 1) + (k + 4 * w) * lda;
    const int bk = lane & 7, bcol = 16 * w + (lane >> 3);
    const double *Ab[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int64_t c = c0 + bcol + 8 * q;
        Ab[q] = A + k + 2 * bk + (c < n ? c : n - 1) * lda;
    }
    double ra[4], rb[2][2];
    auto load = [&] {
#pragma unroll
        for (int q = 0; q < 4; ++q) ra[q] = Aa[q * lda];
        Aa += 16 * lda;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            rb[q][0] = Ab[q][0];
            rb[q][1] = Ab[q][1];
            Ab[q] += 16;
        }
    };
    auto stash = [&](int buf) {
        As[buf][2 * w][lane] = double2{ra[0], ra[1]};
        As[buf][2 * w + 1][lane] = double2{ra[2], ra[3]};
        Bs[buf][bk][bcol] = double2{rb[0][0], rb[0][1]};
        Bs[buf][bk][bcol + 8] = double2{rb[1][0], rb[1][1]};
    };
    d4 acc[2][2];
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J) acc[I][J] = d4_zero();
    load();
    stash(0);
    __syncthreads();
    const int ri = 32 * wi + (lane & 15), rj = 32 * wj + (lane & 15), kq = lane >> 4;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        const int buf = ch & 1;
        if (ch + 1 < NCH) load();
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
        if (ch + 1 < NCH) stash(buf ^ 1);
        __syncthreads();
    }
    d4 c[2][2];
    auto at = [&](int I, int J, int r, bool &ok) {
        const int64_t row = i0 + 32 * wi + 16 * I + d_col(lane), col = c0 + 32 * wj + 16 * J + d_row(r, lane);
        ok = row < m && col < n;
        return ok ? row + col * lda : r0 + r0 * lda;
    };
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                bool ok;
                c[I][J][r] = A[at(I, J, r, ok)];
            }
#pragma unroll
    for (int I = 0; I < 2; ++I)
#pragma unroll
        for (int J = 0; J < 2; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                bool ok;
                const int64_t e = at(I, J, r, ok);
                if (ok) A[e] = c[I][J][r] - acc[I][J][r];
            }
}

}  // namespace

hipError_t launch_calu_clear(int32_t *dinfo, hipStream_t st) {
    hipLaunchKernelGGL(k_calu_clear, dim3(1), dim3(64), 0, st, dinfo);
    return hipGetLastError();
}

hipError_t launch_calu_panel_rest(double *A, int64_t lda, int64_t m, int64_t n, int64_t k, int b,
                                  const int64_t *piv, int32_t *meta, int64_t *ipiv_out, const int32_t *pinfo,
                                  int32_t *dinfo, const double *L, int64_t ldl, const double *U, int64_t ldu,
                                  hipStream_t st) {
    if (b < 1 || b > kLuPanel) return hipErrorInvalidValue;
    {
        ProfScope ps("calu_swaps", st);
        hipLaunchKernelGGL(k_calu_swaps, dim3(1), dim3(64), 0, st, piv, b, k, meta, ipiv_out + k, pinfo, dinfo);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n > b) {
        ProfScope ps("calu_rowswap", st);
        hipLaunchKernelGGL(k_calu_rowswap, dim3((unsigned)((n - b + 3) / 4)), dim3(256), 0, st, A, lda, n, k, b,
                           meta);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    {
        ProfScope ps("calu_pack", st);
        const int64_t mr = m - k;
        hipLaunchKernelGGL(k_calu_pack, dim3((unsigned)((mr + 255) / 256)), dim3(256), 0, st, A, lda, mr, k, b,
                           meta, L, ldl, U, ldu);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (k + b < n) {
        {
            ProfScope ps("calu_trsm", st);
            const int64_t cols = n - k - b;
            hipLaunchKernelGGL(k_calu_trsm, dim3((unsigned)((cols + 15) / 16)), dim3(64), 0, st, A, lda, n, k);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        const int64_t Tr = (m - k - b + 63) / 64, Tc = (n - k - b + 63) / 64;
        if (Tr * Tc > INT32_MAX) return hipErrorInvalidValue;
        ProfScope ps("calu_update", st);
        hipLaunchKernelGGL(k_lu_update, dim3((unsigned)(Tr * Tc)), dim3(256), 0, st, A, lda, m, n, k, Tr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tsqr
