// orth.hip -- block orthogonalisation against an orthonormal basis, the
// step that block-iterative methods (block Krylov solvers, block
// eigensolvers) repeat to grow an orthogonal basis, with TSQR as the stable
// orthogonalisation of each new block (the paper's Scope section and
// Sec. 6: TSQR generates an orthogonal basis for a set of vectors stably,
// with few messages).
//
// For an orthonormal V (m x nv) and a new block W (m x b), two passes of
// block classical Gram-Schmidt
//     H1 = V^T W,  W <- W - V H1,  H2 = V^T W,  W <- W - V H2
// (the second pass restores orthogonality to V lost to rounding in the
// first), then TSQR of the projected W = Q R and Q written over W:
//     W_in = V (H1 + H2) + Q R,   [V Q]^T [V Q] = I.
//
// Kernels (FP64 matrix-core tiles v_mfma_f64_16x16x4f64, layout in mfma.h):
//   k_proj_partial  per row block, the nv x b partial V_blk^T W_blk: wave w
//                   owns 16 columns of a 64-column slice of V, a lane loads 4
//                   consecutive rows of one column (16-byte loads) and feeds
//                   4 matrix-core k-steps;
//   k_proj_stream   the same two products with V read in 16-row tiles that a
//                   wave keeps in registers, for up to 128 columns of V and 32
//                   of W: the first pass' update and the second's V^T W then
//                   share one read of V;
//   k_proj_reduce   H = sum of the partials in block order (deterministic);
//   k_proj_update   W -= V H: a wave owns 16 rows, the k-loop runs over V's
//                   columns 4 at a time; V is read in whole 128-byte row
//                   segments of a column.
#include <type_traits>

#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

namespace {

constexpr int kProjSlice = 64;   // V columns per workgroup of the partial pass

typedef double dv2o __attribute__((ext_vector_type(2)));

// Rows [r, r + 4) of column `col` (zeros past `hi` or past `cols`).
__device__ __forceinline__ void rows4(const double *__restrict__ M, int64_t ld, int64_t r, int64_t hi, int col,
                                      int cols, double (&v)[4]) {
    const bool ok = col < cols;
    const double *p = M + r + (int64_t)(ok ? col : 0) * ld;
    if (ok && r + 4 <= hi && (reinterpret_cast<uintptr_t>(p) & 15) == 0) {
        const dv2o a = *reinterpret_cast<const dv2o *>(p);
        const dv2o b = *reinterpret_cast<const dv2o *>(p + 2);
        v[0] = a.x;
        v[1] = a.y;
        v[2] = b.x;
        v[3] = b.y;
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = (ok && r + q < hi) ? p[q] : 0.0;
    }
}

// Hpart[blk] (nv x b, column-major, ld nv) for columns [64 y, 64 y + 64)
// of V: block blk covers rows [blk per, (blk + 1) per), per a multiple of 16.
__global__ __launch_bounds__(256) void k_proj_partial(const double *__restrict__ V, int64_t ldv, int nv,
                                                      const double *__restrict__ W, int64_t ldw, int b,
                                                      int64_t m, int64_t per, double *__restrict__ Hpart) {
    const int tid = local_tid(), lane = tid & 63, w = tid >> 6;
    const int i = lane & 15, kq = lane >> 4;
    const int c0 = kProjSlice * blockIdx.y + 16 * w;
    const int64_t lo = (int64_t)blockIdx.x * per;
    const int64_t hi = (lo + per < m) ? lo + per : m;
    const int nJ = (b + 15) / 16;
    d4 acc[4];
#pragma unroll
    for (int J = 0; J < 4; ++J) acc[J] = d4_zero();
    if (c0 < nv) {
        for (int64_t r = lo; r < hi; r += 16) {
            // lane (i, kq) holds rows r + 4 kq .. r + 4 kq + 3; k-step s of
            // the tile uses row r + 4 kq + s for k-index kq
            const int64_t rr = r + 4 * kq;
            double a[4];
            rows4(V, ldv, rr, hi, c0 + i, nv, a);
#pragma unroll
            for (int J = 0; J < 4; ++J) {
                if (J < nJ) {
                    double bw[4];
                    rows4(W, ldw, rr, hi, 16 * J + i, b, bw);
#pragma unroll
                    for (int s = 0; s < 4; ++s) acc[J] = mfma_f64(a[s], bw[s], acc[J]);
                }
            }
        }
    }
    double *P = Hpart + (int64_t)blockIdx.x * nv * b;
#pragma unroll
    for (int J = 0; J < 4; ++J) {
        if (J >= nJ) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = c0 + d_row(q, lane), col = 16 * J + d_col(lane);
            if (row < nv && col < b) P[row + (int64_t)col * nv] = acc[J][q];
        }
    }
}

// H = sum over blocks of Hpart, one workgroup per 64 entries (wave w sums
// blocks w, w + 4, ..., the four meet in wave order); if Hacc, also Hacc += H.
// 256 blocks of 96 x 16: 42 -> 8 us against one thread per entry.
__global__ __launch_bounds__(256) void k_proj_reduce(const double *__restrict__ Hpart, int nblk, int nv, int b,
                                                     double *__restrict__ H, int64_t ldh,
                                                     double *__restrict__ Hacc, int64_t ldacc) {
    __shared__ double part[4][64];
    const int lane = threadIdx.x & 63, w = wave_index<4>();
    const int64_t total = (int64_t)nv * b, e = (int64_t)blockIdx.x * 64 + lane;
    const double *p = Hpart + (e < total ? e : 0);
    double s[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] = 0.0;
    for (int q = w; q < nblk; q += 32) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(q + 4 * u < nblk ? q + 4 * u : q) * total];
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] += q + 4 * u < nblk ? v[u] : 0.0;
    }
    part[w][lane] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    __syncthreads();
    if (w == 0 && e < total) {
        const double h = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
        const int r = (int)(e % nv), c = (int)(e / nv);
        H[r + (int64_t)c * ldh] = h;
        if (Hacc) Hacc[r + (int64_t)c * ldacc] += h;
    }
}

// W -= V H (UPD) and / or the partials V^T W of the (updated) W (PART), nv <=
// 16 NT columns of V, b <= 16 NJ of W.  A wave takes 16-row tiles gw, gw + all
// waves, ..., the next tile's loads in flight: V with rows on lanes % 16,
// column 4 c + lane / 16 in register c, which is the operand of the
// (transposed) update as it stands; V^T W contracts the rows, and takes V and
// W with lanes and columns exchanged through the wave's own part of LDS, four
// column tiles at a time.  No barrier between the first and the last tile.
// What bounds it: reading V.  1,048,576 rows, 96 columns of V, 16 of W: three
// passes of 0.21, 0.24 and 0.24 ms (3.1 GB, 4.5 TB/s) against four of 0.33 and
// 0.43 ms with V^T W and V H by kernels that load operands as they use them.
template <int NT, int NJ, int NW>
struct ProjSmem {
    double H[16 * NT][16 * NJ];
    double X[NW][4 + NJ][16][17];   // [wave][tile][column][row]
};
template <int NT, int NJ, int NW, bool UPD, bool PART>
__global__ __launch_bounds__(64 * NW) void k_proj_stream(const double *__restrict__ V, int64_t ldv, int nv,
                                                         const double *__restrict__ H, int64_t ldh,
                                                         double *__restrict__ W, int64_t ldw, int b, int64_t m,
                                                         double *__restrict__ Hpart) {
    extern __shared__ __attribute__((aligned(16))) double smem_raw[];
    ProjSmem<NT, NJ, NW> &sm = *reinterpret_cast<ProjSmem<NT, NJ, NW> *>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index<NW>(), i = lane & 15, kq = lane >> 4;
    double(*X)[16][17] = sm.X[w];
    if constexpr (UPD) {
        for (int e = tid; e < 16 * NT * 16 * NJ; e += 64 * NW) {
            const int k = e / (16 * NJ), c = e % (16 * NJ);
            const double h = H[(k < nv ? k : 0) + (int64_t)(c < b ? c : 0) * ldh];
            sm.H[k][c] = (k < nv && c < b) ? h : 0.0;
        }
    }
    __syncthreads();
    d4 part[NT][NJ];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int J = 0; J < NJ; ++J) part[t][J] = d4_zero();
    double vn[4 * NT], wn[NJ][4];
    // columns past the last repeat it (their products are dropped), rows past
    // the end the last row (zero in W)
    auto fetch = [&](int64_t g) {
        const int64_t row = 16 * g + i < m ? 16 * g + i : m - 1;
        int k = kq;
        // the columns' offsets are kept over the loop only where registers are left
        if constexpr (NT * NJ >= 8) asm volatile("" : "+v"(k));
#pragma unroll
        for (int c = 0; c < 4 * NT; ++c) vn[c] = V[row + (int64_t)(4 * c + k < nv ? 4 * c + k : nv - 1) * ldv];
#pragma unroll
        for (int J = 0; J < NJ; ++J)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = 16 * J + 4 * q + k;
                wn[J][q] = W[row + (int64_t)(c < b ? c : b - 1) * ldw];
            }
    };
    const int64_t groups = (m + 15) / 16, step = (int64_t)gridDim.x * NW;
    int64_t g = (int64_t)blockIdx.x * NW + w;
    fetch(g < groups ? g : groups - 1);
#pragma unroll 1
    for (; g < groups; g += step) {
        double v[4 * NT], wt[NJ][4];
#pragma unroll
        for (int c = 0; c < 4 * NT; ++c) v[c] = vn[c];
#pragma unroll
        for (int J = 0; J < NJ; ++J)
#pragma unroll
            for (int q = 0; q < 4; ++q) wt[J][q] = 16 * g + i < m ? wn[J][q] : 0.0;
        fetch(g + step < groups ? g + step : groups - 1);
        if constexpr (UPD) {
#pragma unroll
            for (int J = 0; J < NJ; ++J) {
                d4 acc = d4_zero();
#pragma unroll
                for (int c = 0; c < 4 * NT; ++c) acc = mfma_f64(sm.H[4 * c + kq][16 * J + i], v[c], acc);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    wt[J][q] -= acc[q];
                    const int c = 16 * J + 4 * q + kq;
                    if (16 * g + i < m && c < b) W[16 * g + i + (int64_t)c * ldw] = wt[J][q];
                }
            }
        }
        if constexpr (PART) {
            double bw[NJ][4];
#pragma unroll
            for (int J = 0; J < NJ; ++J)
#pragma unroll
                for (int q = 0; q < 4; ++q) X[4 + J][4 * q + kq][i] = 16 * g + i < m ? wt[J][q] : 0.0;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int J = 0; J < NJ; ++J)
#pragma unroll
                for (int s = 0; s < 4; ++s) bw[J][s] = X[4 + J][i][4 * s + kq];
#pragma unroll
            for (int t0 = 0; t0 < NT; t0 += 4) {
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (t0 + c / 4 < NT) X[c / 4][4 * (c & 3) + kq][i] = v[4 * t0 + c];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int t = t0; t < t0 + 4 && t < NT; ++t)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const double a = X[t - t0][i][4 * s + kq];
#pragma unroll
                        for (int J = 0; J < NJ; ++J) part[t][J] = mfma_f64(a, bw[J][s], part[t][J]);
                    }
            }
        }
    }
    if constexpr (PART) {
        // the waves' partials in wave order, through LDS
        double *sum = &sm.X[0][0][0][0];   // [tile][register][lane]
        static_assert(NT * NJ * 256 <= NW * (4 + NJ) * 16 * 17, "fits");
        for (int u = 0; u < NW; ++u) {
            __syncthreads();
            if (w == u) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int J = 0; J < NJ; ++J)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            double &x = sum[((t * NJ + J) * 4 + q) * 64 + lane];
                            x = u ? x + part[t][J][q] : part[t][J][q];
                            const int r = 16 * t + d_row(q, lane), c = 16 * J + d_col(lane);
                            if (u == NW - 1 && r < nv && c < b) Hpart[((int64_t)blockIdx.x * b + c) * nv + r] = x;
                        }
            }
        }
    }
}

// W[rows] -= V[rows] H for the 64-row groups g = blockIdx.x, blockIdx.x +
// gridDim.x, ...: wave w takes rows 16 w .. 16 w + 15 of a group.
__global__ __launch_bounds__(256) void k_proj_update(const double *__restrict__ V, int64_t ldv, int nv,
                                                     const double *__restrict__ H, int64_t ldh,
                                                     double *__restrict__ W, int64_t ldw, int b, int64_t m) {
    const int tid = local_tid(), lane = tid & 63, w = tid >> 6;
    const int i = lane & 15, kq = lane >> 4;
    const int nJ = (b + 15) / 16;
    const int64_t groups = (m + 63) / 64;
    for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
        const int64_t r0 = 64 * g + 16 * w;
        if (r0 >= m) continue;
        d4 acc[4];
#pragma unroll
        for (int J = 0; J < 4; ++J) acc[J] = d4_zero();
        const int64_t row = r0 + i;
        const bool rok = row < m;
#pragma unroll 4
        for (int k0 = 0; k0 < nv; k0 += 4) {
            // A[i][kq] = V[r0 + i][k0 + kq], B[kq][j] = H[k0 + kq][16 J + j]
            const int kk = k0 + kq;
            const bool kok = kk < nv;
            const double a = (rok && kok) ? V[row + (int64_t)kk * ldv] : 0.0;
#pragma unroll
            for (int J = 0; J < 4; ++J) {
                if (J < nJ) {
                    const int col = 16 * J + i;
                    const double h = (kok && col < b) ? H[kk + (int64_t)col * ldh] : 0.0;
                    acc[J] = mfma_f64(a, h, acc[J]);
                }
            }
        }
#pragma unroll
        for (int J = 0; J < 4; ++J) {
            if (J >= nJ) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t rw = r0 + d_row(q, lane);
                const int col = 16 * J + d_col(lane);
                if (rw < m && col < b) W[rw + (int64_t)col * ldw] -= acc[J][q];
            }
        }
    }
}

}  // namespace

int proj_blocks(int64_t m) {
    // rows per block a multiple of 16, about 4096 rows per block, at most
    // kProjMaxBlocks blocks
    int64_t nb = (m + 4095) / 4096;
    if (nb > kProjMaxBlocks) nb = kProjMaxBlocks;
    return (int)(nb < 1 ? 1 : nb);
}

// The streaming form's workgroups: 8 waves where two a SIMD fit its registers
// (NT NJ <= 8), else 4; one per compute unit, fewer where a wave would have no
// tile; where partials are kept, no more than `slots` of them (one for about
// 4,096 rows).
template <int NT, int NJ, bool UPD, bool PART>
static hipError_t proj_stream(const double *V, int64_t ldv, int nv, const double *H, int64_t ldh, double *W,
                              int64_t ldw, int b, int64_t m, double *Hpart, int64_t slots, int *nblk,
                              hipStream_t st) {
    constexpr int NW = NT * NJ <= 8 ? 8 : 4;
    const size_t sh = sizeof(ProjSmem<NT, NJ, NW>);
    const auto kern = k_proj_stream<NT, NJ, NW, UPD, PART>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    const int64_t full = kComputeUnits, need = (m + 16 * NW - 1) / (16 * NW);
    int64_t grid = need < full ? need : full;
    if (PART && grid > slots) grid = slots;
    if (nblk) *nblk = (int)grid;
    ProfScope ps(UPD ? (PART ? "orth_proj_both" : "orth_proj_update") : "orth_proj_partial", st);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW), sh, st, V, ldv, nv, H, ldh, W, ldw, b, m, Hpart);
    return hipGetLastError();
}
template <bool UPD, bool PART>
static hipError_t proj_stream(const double *V, int64_t ldv, int nv, const double *H, int64_t ldh, double *W,
                              int64_t ldw, int b, int64_t m, double *Hpart, int64_t slots, int *nblk,
                              hipStream_t st) {
    auto go = [&](auto nt, auto nj) {
        return proj_stream<decltype(nt)::value, decltype(nj)::value, UPD, PART>(V, ldv, nv, H, ldh, W, ldw, b, m,
                                                                                Hpart, slots, nblk, st);
    };
    auto with_nj = [&](auto nt) {
        return b <= 16 ? go(nt, std::integral_constant<int, 1>{}) : go(nt, std::integral_constant<int, 2>{});
    };
    if (nv <= 16) return with_nj(std::integral_constant<int, 1>{});
    if (nv <= 32) return with_nj(std::integral_constant<int, 2>{});
    if (nv <= 64) return with_nj(std::integral_constant<int, 4>{});
    if (nv <= 96) return with_nj(std::integral_constant<int, 6>{});
    return with_nj(std::integral_constant<int, 8>{});
}

static hipError_t proj_reduce(const double *Hpart, int nblk, int nv, int b, double *H, int64_t ldh, double *Hacc,
                              int64_t ldacc, hipStream_t st) {
    ProfScope ps("orth_proj_reduce", st);
    const int64_t total = (int64_t)nv * b;
    hipLaunchKernelGGL(k_proj_reduce, dim3((unsigned)((total + 63) / 64)), dim3(256), 0, st, Hpart, nblk, nv, b, H,
                       ldh, Hacc, ldacc);
    return hipGetLastError();
}

static hipError_t proj_partial(const double *V, int64_t ldv, int nv, const double *W, int64_t ldw, int b, int64_t m,
                               double *Hpart, int *nblk, hipStream_t st) {
    *nblk = proj_blocks(m);
    const int64_t per = ((m + *nblk - 1) / *nblk + 15) / 16 * 16;
    ProfScope ps("orth_proj_partial", st);
    hipLaunchKernelGGL(k_proj_partial, dim3((unsigned)*nblk, (unsigned)((nv + kProjSlice - 1) / kProjSlice)),
                       dim3(256), 0, st, V, ldv, nv, W, ldw, b, m, per, Hpart);
    return hipGetLastError();
}

static hipError_t proj_update(const double *V, int64_t ldv, int nv, const double *H, int64_t ldh, double *W,
                              int64_t ldw, int b, int64_t m, hipStream_t st) {
    ProfScope ps("orth_proj_update", st);
    const int64_t groups = (m + 63) / 64;
    const unsigned grid = (unsigned)(groups < 2048 ? groups : 2048);
    hipLaunchKernelGGL(k_proj_update, dim3(grid), dim3(256), 0, st, V, ldv, nv, H, ldh, W, ldw, b, m);
    return hipGetLastError();
}

// Two passes of block classical Gram-Schmidt: W -= V H1, W -= V H2, H = H1 +
// H2.  The streaming kernel holds a 16-row tile of V and the partials in
// registers: up to 128 columns of V and 32 of W; wider ones read V by slices.
hipError_t launch_cgs2(const double *V, int64_t ldv, int nv, double *W, int64_t ldw, int b, int64_t m,
                       double *Hpart, double *H, int64_t ldh, double *H2, hipStream_t st) {
#define CGS_TRY(x)                        \
    do {                                  \
        const hipError_t e_ = (x);        \
        if (e_ != hipSuccess) return e_;  \
    } while (0)
    int nblk = 0;
    const bool stream = nv <= 128 && b <= 32;
    const int64_t slots = proj_blocks(m);
    if (stream)
        CGS_TRY((proj_stream<false, true>(V, ldv, nv, nullptr, 0, W, ldw, b, m, Hpart, slots, &nblk, st)));
    else
        CGS_TRY(proj_partial(V, ldv, nv, W, ldw, b, m, Hpart, &nblk, st));
    CGS_TRY(proj_reduce(Hpart, nblk, nv, b, H, ldh, nullptr, 0, st));
    if (stream) {
        CGS_TRY((proj_stream<true, true>(V, ldv, nv, H, ldh, W, ldw, b, m, Hpart, slots, &nblk, st)));
    } else {
        CGS_TRY(proj_update(V, ldv, nv, H, ldh, W, ldw, b, m, st));
        CGS_TRY(proj_partial(V, ldv, nv, W, ldw, b, m, Hpart, &nblk, st));
    }
    CGS_TRY(proj_reduce(Hpart, nblk, nv, b, H2, nv, H, ldh, st));
    if (stream) return proj_stream<true, false>(V, ldv, nv, H2, nv, W, ldw, b, m, nullptr, 0, nullptr, st);
    return proj_update(V, ldv, nv, H2, nv, W, ldw, b, m, st);
#undef CGS_TRY
}

}  // namespace tsqr
