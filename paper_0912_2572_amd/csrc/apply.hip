// apply.hip -- applying the TSQR orthogonal factor to a block of columns.
//
// Q is the product of the leaf factors (one per chunk of every domain) and
// the tree factors (one per combine), each in compact-WY form
// I - Y T Y^T (Sec. 2.2).  Q^T B runs the leaves first, chunk by chunk in
// factorization order, then the tree bottom-up; Q B runs the same pieces in
// the reverse order with T in place of T^T (Sec. 2.3: the tree that reduced
// R is reused for Q, Property 1 of Sec. 4).
//
// A chunk k >= 1 of a domain has Y = [I; V_k] on the rows [domain top n rows;
// chunk rows], so with the n-row block Yb (the domain's top rows of B):
//     W = Yb + V_k^T B_k,  W <- T_k^T W (or T_k W),  Yb -= W,  B_k -= V_k W.
// The first chunk of a domain has a plain unit-lower-trapezoidal V_0.
// A tree node (l, r) has Y = [I; U] with U the n x n upper triangle stored
// in the right child's slot, acting on the top n rows of domains l and r.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

namespace {

constexpr int KB = 16;   // columns of B per workgroup: one matrix-core tile

// 16 x 16 tiles (t, c), t <= c, of an upper triangle: tile_at(t, c) is the
// tile's place.  Rows are 17 apart: both operand orders read without bank
// conflicts.
constexpr int kTileLd = 17;
__host__ __device__ constexpr int tile_at(int t, int c) { return c * (c + 1) / 2 + t; }

template <int NT>
struct TreeApplySmem {
    double U[NT * (NT + 1) / 2][16][kTileLd];
    double T[NT * (NT + 1) / 2][16][kTileLd];
    double YZ[16 * NT][kTileLd];   // the right's block, then Z
    double W[16 * NT][kTileLd];
};
static_assert(2 * sizeof(TreeApplySmem<4>) <= 160 * 1024, "two workgroups per CU");

// Wave W's part of a node: rows 16 W .. 16 W + 15 of each product; y: those
// rows of the left's block, yr (out): of the right's.
template <bool QT, int NT, int W>
__device__ __forceinline__ void tree_apply_node(TreeApplySmem<NT> &sm, d4 &y, d4 &yr) {
    constexpr int T0 = QT ? 0 : W, T1 = QT ? W : NT - 1;   // T's tiles
    const int lane = threadIdx.x & 63, cg = lane & 15, rg = lane >> 4;
    d4 acc = y;
#pragma unroll
    for (int t = 0; t <= W; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double b = sm.YZ[16 * t + 4 * u + rg][cg];
            if (t == W) yr[u] = b;
            acc = mfma_f64(sm.U[tile_at(t, W)][4 * u + rg][cg], b, acc);
        }
#pragma unroll
    for (int u = 0; u < 4; ++u) sm.W[16 * W + 4 * u + rg][cg] = acc[u];
    __syncthreads();
    acc = d4_zero();
#pragma unroll
    for (int t = T0; t <= T1; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double a = QT ? sm.T[tile_at(t, W)][4 * u + rg][cg] : sm.T[tile_at(W, t)][cg][4 * u + rg];
            acc = mfma_f64(a, sm.W[16 * t + 4 * u + rg][cg], acc);
        }
    y -= acc;
#pragma unroll
    for (int u = 0; u < 4; ++u) sm.YZ[16 * W + 4 * u + rg][cg] = acc[u];
    __syncthreads();
#pragma unroll
    for (int t = W; t < NT; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            yr = mfma_f64(-sm.U[tile_at(W, t)][cg][4 * u + rg], sm.YZ[16 * t + 4 * u + rg][cg], yr);
}

// One chain of the tree for the 16-column block cblk of B: the chain's nodes
// (left, right) in order (Q^T) or in reverse order (Q).  Wave w owns rows
// 16 w .. 16 w + 15 of the left's block (in registers throughout) and of every
// n-row product, all three of them 16 x 16 x 4 matrix-core tiles:
//     W = Yl + U^T Yr,   Z = T^T W or T W,   Yl -= Z,   Yr -= U Z.
// The next node's U, T and Yr are read (a column per wave and load: 512
// consecutive bytes) into registers while a node runs, and pass to the
// operand layouts through LDS.  What bounds it: latency, under a launch per
// level.  Measured at n = 64 against a dot product per thread on operands in
// LDS: one column, a level of a 256-domain tree 13.5 -> 8.5 us; 448 columns,
// the level of 128 chains 247 -> 73 us (36 tiles of 64 cycles a wave and block
// are 12 us of that, the rest is the loads').  Loading the operands straight
// into their layouts was slower (88 us: 16 lines an instruction).
template <bool QT, int NT>
__device__ __forceinline__ void tree_apply_chain(TreeApplySmem<NT> &sm, const double *__restrict__ Rdom,
                                                 const double *__restrict__ Tnode, const PanelArgs &pa,
                                                 int64_t left, int64_t stride, int64_t span,
                                                 double *__restrict__ B, int64_t ldb, int64_t k, int64_t cblk) {
    const int n = pa.n;
    const int64_t nn = (int64_t)n * n, c0 = cblk * KB;
    const int kc = (int)((k - c0 < KB) ? k - c0 : KB);
    const int w = wave_index<4>(), lane = threadIdx.x & 63, cg = lane & 15, rg = lane >> 4;
    int64_t nr = 0;
    for (int64_t q = 1; q * stride < span && left + q * stride < pa.P; ++q) ++nr;
    double *B0 = B + c0 * ldb;
    double uv[4 * NT], tv[4 * NT], yv[4];
    auto fetch = [&](int64_t right) {
        const double *U = Rdom + right * nn;
        const double *T = Tnode + right * nn;
        const double *Yr = B0 + dom_row0(pa, right) + (lane < n ? lane : 0);
#pragma unroll
        for (int u = 0; u < 4 * NT; ++u) {
            const int c = w + 4 * u, e = (lane <= c && c < n) ? lane + c * n : 0;
            uv[u] = U[e];
            tv[u] = T[e];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) yv[u] = Yr[(4 * w + u < kc ? 4 * w + u : 0) * ldb];
    };
    auto right_of = [&](int64_t qq) { return left + (QT ? qq + 1 : nr - qq) * stride; };
    if (nr > 0) fetch(right_of(0));
    double *Yl = B0 + dom_row0(pa, left) + (cg < kc ? cg : 0) * ldb;
    d4 y = d4_zero(), yr = d4_zero();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int row = 16 * w + 4 * u + rg;
        const double v = Yl[row < n ? row : 0];
        y[u] = (cg < kc && row < n) ? v : 0.0;
    }
#pragma unroll 1
    for (int64_t qq = 0; qq < nr; ++qq) {
#pragma unroll
        for (int u = 0; u < 4 * NT; ++u) {
            const int c = w + 4 * u, tc = u >> 2;
            const bool ok = lane <= c && c < n;
            if ((lane >> 4) <= tc) {
                sm.U[tile_at(0, tc) + (lane >> 4)][cg][c & 15] = ok ? uv[u] : 0.0;
                sm.T[tile_at(0, tc) + (lane >> 4)][cg][c & 15] = ok ? tv[u] : 0.0;
            }
        }
        if (lane < 16 * NT) {
#pragma unroll
            for (int u = 0; u < 4; ++u) sm.YZ[lane][4 * w + u] = (lane < n && 4 * w + u < kc) ? yv[u] : 0.0;
        }
        __syncthreads();
        if (qq + 1 < nr) fetch(right_of(qq + 1));
        switch (w) {
            case 0: tree_apply_node<QT, NT, 0>(sm, y, yr); break;
            case 1: if constexpr (NT > 1) { tree_apply_node<QT, NT, 1>(sm, y, yr); break; } [[fallthrough]];
            case 2: if constexpr (NT > 2) { tree_apply_node<QT, NT, 2>(sm, y, yr); break; } [[fallthrough]];
            case 3: if constexpr (NT > 3) { tree_apply_node<QT, NT, 3>(sm, y, yr); break; } [[fallthrough]];
            default: __syncthreads(); __syncthreads();
        }
        double *Yr = B0 + dom_row0(pa, right_of(qq)) + (cg < kc ? cg : 0) * ldb;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int row = 16 * w + 4 * u + rg;
            if (cg < kc && row < n) Yr[row] = yr[u];
        }
        if (qq + 1 < nr) __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int row = 16 * w + 4 * u + rg;
        if (cg < kc && row < n) Yl[row] = y[u];
    }
}

}  // namespace

// Tree level: chain g combines rights into left; the Y blocks are the top n
// rows of the domains involved.
template <bool QT, int NT>
__global__ __launch_bounds__(256, 2) void k_tree_apply(const double *__restrict__ Rdom,
                                                    const double *__restrict__ Tnode, PanelArgs pa,
                                                    TreeArgs ta, double *__restrict__ B, int64_t ldb,
                                                    int64_t k) {
    extern __shared__ __attribute__((aligned(16))) double smem_raw[];
    TreeApplySmem<NT> &sm = *reinterpret_cast<TreeApplySmem<NT> *>(smem_raw);
    // A latency-bound chain that may share CUs with a thin Q's top-down tree:
    // its waves take the issue slots first.
    __builtin_amdgcn_s_setprio(3);
    const int64_t left = tree_left(ta, blockIdx.x);
    if (left >= pa.P) return;
    tree_apply_chain<QT, NT>(sm, Rdom, Tnode, pa, left, ta.stride, ta.span, B, ldb, k, blockIdx.y);
}

// Batched: level `step` from the bottom (Q^T) or from the top (Q) of each
// listed matrix's own tree, on its vector F.
template <bool QT>
__global__ __launch_bounds__(256, 2) void k_tree_apply_b(const BMat *__restrict__ mats,
                                                      const int *__restrict__ list, int step, int sweep) {
    extern __shared__ __attribute__((aligned(16))) double smem_raw[];
    const BMat &M = mats[list[blockIdx.y]];
    if (step >= M.nlev) return;
    if (sweep > 0 && M.status[1]) return;
    const TreeArgs ta = M.lev[QT ? step : M.nlev - 1 - step];
    if ((int64_t)blockIdx.x >= ta.chains) return;
    const int64_t left = tree_left(ta, blockIdx.x);
    if (left >= M.pa.P) return;
    auto run = [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        tree_apply_chain<QT, NT>(*reinterpret_cast<TreeApplySmem<NT> *>(smem_raw), M.Rdom, M.Tnode, M.pa, left,
                                 ta.stride, ta.span, M.F, M.pa.m, 1, 0);
    };
    switch ((M.pa.n + 15) >> 4) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        default: run(std::integral_constant<int, 4>{});
    }
}

__global__ void k_scale_b(const BMat *__restrict__ mats, const int *__restrict__ list, int sweep) {
    const BMat &M = mats[list[blockIdx.x]];
    if (sweep > 0 && M.status[1]) return;
    for (int r = threadIdx.x; r < M.pa.n; r += blockDim.x) M.F[r] *= M.dsign[r];
}

__global__ void k_scale_rows(double *B, int64_t ldb, int n, int64_t k, const double *d) {
    for (int64_t e = threadIdx.x + (int64_t)blockIdx.x * blockDim.x; e < (int64_t)n * k;
         e += (int64_t)blockDim.x * gridDim.x) {
        const int r = (int)(e % n);
        const int64_t c = e / n;
        B[r + c * ldb] *= d[r];
    }
}

template <int NT>
static hipError_t tree_apply(const double *Rdom, const double *Tnode, const PanelArgs &pa, const TreeArgs &ta,
                             double *B, int64_t ldb, int64_t k, int trans, hipStream_t st) {
    const size_t sh = sizeof(TreeApplySmem<NT>);
    const auto kern = trans ? k_tree_apply<true, NT> : k_tree_apply<false, NT>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)ta.chains, (unsigned)((k + KB - 1) / KB));
    ProfScope ps(trans ? "tree_apply_qt" : "tree_apply_q", st);
    hipLaunchKernelGGL(kern, grid, dim3(256), sh, st, Rdom, Tnode, pa, ta, B, ldb, k);
    return hipGetLastError();
}

hipError_t launch_tree_apply(const double *Rdom, const double *Tnode, const PanelArgs &pa,
                             const TreeArgs &ta, double *B, int64_t ldb, int64_t k, int trans,
                             hipStream_t st) {
    if (k <= 0) return hipSuccess;
    switch ((pa.n + 15) >> 4) {
        case 1: return tree_apply<1>(Rdom, Tnode, pa, ta, B, ldb, k, trans, st);
        case 2: return tree_apply<2>(Rdom, Tnode, pa, ta, B, ldb, k, trans, st);
        case 3: return tree_apply<3>(Rdom, Tnode, pa, ta, B, ldb, k, trans, st);
        default: return tree_apply<4>(Rdom, Tnode, pa, ta, B, ldb, k, trans, st);
    }
}

hipError_t launch_scale_rows(double *B, int64_t ldb, int n, int64_t k, const double *d, hipStream_t st) {
    if (k <= 0) return hipSuccess;
    ProfScope ps("scale_rows", st);
    hipLaunchKernelGGL(k_scale_rows, dim3(8), dim3(256), 0, st, B, ldb, n, k, d);
    return hipGetLastError();
}

hipError_t launch_tree_apply_b(const BMat *mats, const int *list, int cnt, int64_t gx, int trans, int step,
                               int sweep, hipStream_t st) {
    if (cnt <= 0 || gx <= 0) return hipSuccess;
    const size_t sh = sizeof(TreeApplySmem<4>);
    const auto kern = trans ? k_tree_apply_b<true> : k_tree_apply_b<false>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    ProfScope ps(trans ? "batch_tree_apply_qt" : "batch_tree_apply_q", st);
    hipLaunchKernelGGL(kern, dim3((unsigned)gx, (unsigned)cnt), dim3(256), sh, st, mats, list, step, sweep);
    return hipGetLastError();
}

hipError_t launch_scale_b(const BMat *mats, const int *list, int cnt, int sweep, hipStream_t st) {
    if (cnt <= 0) return hipSuccess;
    ProfScope ps("batch_scale_rows", st);
    hipLaunchKernelGGL(k_scale_b, dim3((unsigned)cnt), dim3(64), 0, st, mats, list, sweep);
    return hipGetLastError();
}

}  // namespace tsqr
