// tree.hip -- tree kernels of the TSQR factorization on gfx950 (Sec. 2.3):
// the structured QR of [R_l; R_r] on the domain triangles, one launch per
// tree level, one workgroup per chain of combines.  The right child's
// triangle is overwritten by the combine's reflector block and its T is
// stored under the right child's index; then the root's R is sign-normalised.
//
// A combine is the panel QR of panel_qr.h with the columns dealt to waves:
// wave w holds columns 16 w .. 16 w + 15 of the right triangle, all its rows,
// and runs its panel's column steps alone, with no barrier and no exchange
// between waves; it then publishes the panel's V and T in LDS and every later
// wave updates its own columns on the matrix cores.  A level is bound by the
// chain of n such steps.  A wave needs a quarter of the registers that one
// wave for the whole triangle would, so that its workgroup finds room beside
// a solve's leaf passes.  k_tree_t builds the parts of T above its diagonal
// blocks after the last level, off the chain of dependent levels.
// A level of one combine: 27 us at 64 columns, 7 at 16 (47 and 12 with every
// step working on all columns behind a barrier).  Other splits measured at 64
// columns: one wave for the whole triangle 34 us, and 95 - 135 beside the
// passes (256 registers a wave wait for half a SIMD to run dry); the rows
// dealt to four waves 33.
#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

namespace {

typedef double dv2 __attribute__((ext_vector_type(2)));

// LDS of a combine of NS column slots.
template <int NS>
struct TreeSmem {
    static constexpr int kLd = 16 * NS + 1, kVtLd = 16 * NS + 4;
    alignas(32) double R[16 * NS * kLd];                 // the left triangle, row-major
    alignas(32) double vt[NS > 1 ? (NS - 1) * 16 * kVtLd : 1];   // V of the panels by columns
    double Tp[NS > 1 ? (NS - 1) * 16 * 17 : 1];             // T of the panels
};

// Column slot w of the upper triangle of an n x n column-major block (tile a:
// rows 16 a .. 16 a + 15), zeros elsewhere.
template <int NS>
__device__ __forceinline__ void load_slot(d4 (&c)[NS], const double *__restrict__ src, int n, int w) {
    const int lane = threadIdx.x & 63, cg = lane & 15, rg = lane >> 4, k = 16 * w + cg;
    const bool vec = (n % 2) == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0;
    const double *p = src + (k < n ? k * n : 0);
#pragma unroll
    for (int a = 0; a < NS; ++a) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = 16 * a + 8 * h + 2 * rg;
            if (vec) {
                const dv2 v = *reinterpret_cast<const dv2 *>(p + (row < n ? row : 0));
                c[a][2 * h] = v.x;
                c[a][2 * h + 1] = v.y;
            } else {
                c[a][2 * h] = p[row < n ? row : 0];
                c[a][2 * h + 1] = p[row + 1 < n ? row + 1 : 0];
            }
        }
    }
#pragma unroll
    for (int a = 0; a < NS; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) c[a][r] = (k < n && 16 * a + tile_row(r, rg) <= k) ? c[a][r] : 0.0;
}

// QR of [R; c] with R in sm.R.  On exit c holds the reflector columns, R
// the new triangle; V and, if T is not null, the panels' T go to memory.
template <int NS>
__device__ __forceinline__ void combine(TreeSmem<NS> &sm, d4 (&c)[NS], const int n, double *__restrict__ V,
                                        double *__restrict__ T) {
    constexpr int LD = TreeSmem<NS>::kLd, VL = TreeSmem<NS>::kVtLd;
    const int lane = threadIdx.x & 63, w = wave_index<NS>(), cg = lane & 15, rg = lane >> 4;
    const int np = (n + 15) >> 4;
    const bool vec = (n % 2) == 0 && (reinterpret_cast<uintptr_t>(V) & 15) == 0;
#pragma unroll 1
    for (int p = 0; p < np; ++p) {
        double *vt = sm.vt + p * 16 * VL, *Tp = sm.Tp + p * 16 * 17;
        if (w == p) {
            PanelRegs pr;
            panel_begin(pr);
#pragma unroll
            for (int a = 0; a < NS; ++a) settle(c[a]);
            auto none = [](auto) {};
            double *Rp = sm.R + 16 * p * (LD + 1);   // the panel's diagonal block of R
            PanelStep<1, NS, false, 0>::run(c, pr, sm, Rp, LD, false, w, rg, cg, none);
            if (n - 16 * p > 8) PanelStep<1, NS, false, 8>::run(c, pr, sm, Rp, LD, false, w, rg, cg, none);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (cg >= 4 * u + rg) Rp[(4 * u + rg) * LD + cg] = pr.rrow[u];
#pragma unroll
            for (int a = 0; a < NS; ++a) c[a] *= pr.scale;
            if (p + 1 < np) {
#pragma unroll
                for (int a = 0; a < NS; ++a) *reinterpret_cast<d4 *>(vt + cg * VL + 16 * a + 4 * rg) = c[a];
                if (rg == 0) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) Tp[cg * 17 + q] = pr.trow[q];
                }
            }
            const int k = 16 * p + cg;
            if (k < n) {
#pragma unroll
                for (int a = 0; a < NS; ++a) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        // (rows past the diagonal tile stay the zeros they are)
                        const int row = 16 * a + 8 * h + 2 * rg;
                        double *d = V + k * n + row;
                        if (vec) {
                            const dv2 x = {c[a][2 * h], c[a][2 * h + 1]};
                            if (a <= p && row < n) *reinterpret_cast<dv2 *>(d) = x;
                        } else {
                            if (a <= p && row < n) d[0] = c[a][2 * h];
                            if (a <= p && row + 1 < n) d[1] = c[a][2 * h + 1];
                        }
                    }
                }
                if (T != nullptr && rg == 0) {
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (16 * p + j < n) T[k + (16 * p + j) * n] = pr.trow[j];
                }
            }
        }
        if constexpr (NS > 1) {
            __syncthreads();
            if (w > p && w < np) {
                // W = V^T C, M = T^T (R rows + W), R rows -= M, C -= V M
                double *Rr = sm.R + 16 * p * LD + 16 * w;
                d4 ev, acc = d4_zero(), mm = d4_zero();
                double ta[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    ev[r] = Rr[(4 * r + rg) * LD + cg];
                    ta[r] = -Tp[(4 * r + rg) * 17 + cg];
                }
#pragma unroll
                for (int a = 0; a < NS; ++a) {
                    if (a > p) continue;
                    const d4 v = *reinterpret_cast<const d4 *>(vt + cg * VL + 16 * a + 4 * rg);
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc = mfma_f64(v[r], c[a][r], acc);
                }
                const d4 wf = acc + ev;
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) mm = mfma_f64(ta[kb], wf[kb], mm);
#pragma unroll
                for (int r = 0; r < 4; ++r) Rr[(4 * r + rg) * LD + cg] = ev[r] + mm[r];
#pragma unroll
                for (int a = 0; a < NS; ++a) {
                    if (a > p) continue;
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb)
                        c[a] = mfma_f64(vt[(4 * kb + rg) * VL + 16 * a + 4 * (cg & 3) + (cg >> 2)], mm[kb], c[a]);
                }
            }
        }
    }
}

// One chain of combines (step 3): left <- qr([R_left; R_right]) for every
// right = left + q stride (q = 1, 2, ... while q stride < span and right < P),
// in order.  The right triangle is overwritten by the combine's reflector
// block V (upper triangular) and, if keep_q, the diagonal blocks of the
// node's T slot by the panels' T.
template <int NS>
__device__ __forceinline__ void tree_chain(TreeSmem<NS> &sm, double *__restrict__ Rdom, double *__restrict__ Tnode,
                                           const PanelArgs &pa, int64_t left, int64_t stride, int64_t span,
                                           int keep_q) {
    constexpr int C = 16 * NS, LD = TreeSmem<NS>::kLd;
    constexpr int S = 64 * NS / C, PASSES = C / S;   // columns a pass over the triangle covers, passes
    const int n = pa.n, w = wave_index<NS>();
    const int64_t nn = (int64_t)n * n;
    if (!(stride < span && left + stride < pa.P)) return;
    d4 c[NS];
    load_slot<NS>(c, Rdom + (left + stride) * nn, n, w);
    const int r = threadIdx.x % C, k0 = threadIdx.x / C;
    {
        // the left triangle, zeros below it and past n; every load in flight
        // before the LDS stores
        const double *p = Rdom + left * nn + (r < n ? r : 0);
        double v[PASSES];
#pragma unroll
        for (int u = 0; u < PASSES; ++u) v[u] = p[(k0 + S * u < n ? k0 + S * u : 0) * n];
#pragma unroll
        for (int u = 0; u < PASSES; ++u) {
            const int k = k0 + S * u;
            sm.R[r * LD + k] = (r <= k && k < n) ? v[u] : 0.0;
        }
    }
    __syncthreads();
    for (int64_t q = 1; q * stride < span; ++q) {
        const int64_t right = left + q * stride;
        if (right >= pa.P) break;
        if (q > 1) load_slot<NS>(c, Rdom + right * nn, n, w);
        combine<NS>(sm, c, n, Rdom + right * nn, keep_q ? Tnode + right * nn : nullptr);
        __syncthreads();
    }
    if (r < n) {
        double *p = Rdom + left * nn + r;
        double v[PASSES];
#pragma unroll
        for (int u = 0; u < PASSES; ++u) v[u] = sm.R[r * LD + k0 + S * u];
#pragma unroll
        for (int u = 0; u < PASSES; ++u) {
            const int k = k0 + S * u;
            if (k < n) p[k * n] = (r <= k) ? v[u] : 0.0;
        }
    }
}

// A node's T above its diagonal blocks (16-column panels t < p), from its
// reflector block V (upper triangular) and the panels' T: with G_tp = V_t^T
// V_p, T[0:16p, p] = -T[0:16p, 0:16p] (G[0:16p, p] T_pp); block row t by wave
// t.  Zeros below the diagonal.
constexpr int kNodeThreads = 256;
struct NodeTSmem {
    double V[64 * 65];   // row-major
    double T[64 * 65];
    double P[48 * 16];
};
__device__ __forceinline__ void node_t(NodeTSmem &sm, const double *__restrict__ V, double *__restrict__ T, int n) {
    constexpr int LD = 65;
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index<4>(), cg = lane & 15, rg = lane >> 4;
    const int np = (n + 15) >> 4, r = lane;
    {
        // wave w: columns w, w + 4, ..., a row per lane; every load in flight
        double v[16], t[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int k = w + 4 * u;
            const int64_t e = (r < n && k < n) ? r + (int64_t)k * n : 0;
            v[u] = V[e];
            t[u] = T[e];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int k = w + 4 * u;
            const bool in = r <= k && k < n;
            sm.V[r * LD + k] = in ? v[u] : 0.0;
            sm.T[r * LD + k] = (in && (r >> 4) == (k >> 4)) ? t[u] : 0.0;
        }
    }
    __syncthreads();
    for (int p = 1; p < np; ++p) {
        if (w < p) {
            // (V_p^T V_t)[i][k] = G[k][i]: the left operand of G T_pp as it stands
            d4 g = d4_zero(), pg = d4_zero();
            for (int kb = 0; kb < 4 * (w + 1); ++kb) {
                const int row = 4 * kb + rg;
                g = mfma_f64(sm.V[row * LD + 16 * p + cg], sm.V[row * LD + 16 * w + cg], g);
            }
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) pg = mfma_f64(g[kb], sm.T[(16 * p + 4 * kb + rg) * LD + 16 * p + cg], pg);
#pragma unroll
            for (int u = 0; u < 4; ++u) sm.P[(16 * w + 4 * u + rg) * 16 + cg] = pg[u];
        }
        __syncthreads();
        if (w < p) {
            d4 acc = d4_zero();
            for (int kb = 4 * w; kb < 4 * p; ++kb) {
                const int k = 4 * kb + rg;
                acc = mfma_f64(sm.T[(16 * w + cg) * LD + k], sm.P[k * 16 + cg], acc);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) sm.T[(16 * w + 4 * u + rg) * LD + 16 * p + cg] = -acc[u];
        }
        __syncthreads();
    }
    if (r < n) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int k = w + 4 * u;
            if (k < n) T[r + (int64_t)k * n] = sm.T[r * LD + k];
        }
    }
}

}  // namespace

// Every tree node's T: nodes 1 .. P - 1 (each domain but 0 is absorbed as
// the right operand of exactly one combine, whatever the tree's shape).
__global__ __launch_bounds__(kNodeThreads) void k_tree_t(const double *__restrict__ Rdom, double *__restrict__ Tnode,
                                                         PanelArgs pa) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    NodeTSmem &sm = *reinterpret_cast<NodeTSmem *>(smem_raw);
    const int64_t node = 1 + (int64_t)blockIdx.x;
    if (node >= pa.P) return;
    const int64_t off = node * (int64_t)pa.n * pa.n;
    node_t(sm, Rdom + off, Tnode + off, pa.n);
}

template <int NS>
__global__ __launch_bounds__(64 * NS) __attribute__((amdgpu_waves_per_eu(2, 4)))
void k_tree(double *__restrict__ Rdom, double *__restrict__ Tnode, PanelArgs pa, TreeArgs ta, int keep_q) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    TreeSmem<NS> &sm = *reinterpret_cast<TreeSmem<NS> *>(smem_raw);
    // The levels are the critical path while a solve's leaf passes share the
    // CUs: the chain's wave takes the issue slots first.
    __builtin_amdgcn_s_setprio(3);
    const int64_t left = tree_left(ta, blockIdx.x);
    if (left >= pa.P) return;
    tree_chain<NS>(sm, Rdom, Tnode, pa, left, ta.stride, ta.span, keep_q);
}

// R_out = D R_root with D = diag(sgn R_jj), sgn(0) = +1; d_out = diag(D).
__global__ void k_sign_normalise(const double *__restrict__ Rroot, int n, double *__restrict__ Rout,
                                 int64_t ldr, int row_off, int col_off, double *__restrict__ dsign) {
    for (int e = threadIdx.x + blockIdx.x * blockDim.x; e < n * n; e += blockDim.x * gridDim.x) {
        const int r = e % n, k = e / n;
        const double dr = (Rroot[r + r * n] < 0.0) ? -1.0 : 1.0;
        Rout[(row_off + r) + (int64_t)(col_off + k) * ldr] = (r <= k) ? dr * Rroot[e] : 0.0;
        if (k == 0) dsign[row_off + r] = dr;
    }
}

// ---- batched forms: grid.y walks the matrix list, grid.x the chains of the
// listed matrix (a workgroup past its matrix's count returns).
template <int NS>
__global__ __launch_bounds__(64 * NS) __attribute__((amdgpu_waves_per_eu(2, 4)))
void k_tree_b(const BMat *__restrict__ mats, const int *__restrict__ list, int level) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    TreeSmem<NS> &sm = *reinterpret_cast<TreeSmem<NS> *>(smem_raw);
    const BMat &M = mats[list[blockIdx.y]];
    if (level >= M.nlev) return;
    const TreeArgs ta = M.lev[level];
    if ((int64_t)blockIdx.x >= ta.chains) return;
    const int64_t left = tree_left(ta, blockIdx.x);
    if (left >= M.pa.P) return;
    tree_chain<NS>(sm, M.Rdom, M.Tnode, M.pa, left, ta.stride, ta.span, 1);
}

__global__ __launch_bounds__(kNodeThreads) void k_tree_t_b(const BMat *__restrict__ mats,
                                                           const int *__restrict__ list) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    NodeTSmem &sm = *reinterpret_cast<NodeTSmem *>(smem_raw);
    const BMat &M = mats[list[blockIdx.y]];
    const int64_t node = 1 + (int64_t)blockIdx.x;
    if (node >= M.pa.P) return;
    const int64_t off = node * (int64_t)M.pa.n * M.pa.n;
    node_t(sm, M.Rdom + off, M.Tnode + off, M.pa.n);
}

__global__ void k_sign_b(const BMat *__restrict__ mats, const int *__restrict__ list) {
    const BMat &M = mats[list[blockIdx.x]];
    const int n = M.pa.n;
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
        const int r = e % n, k = e / n;
        const double dr = (M.Rdom[r + r * n] < 0.0) ? -1.0 : 1.0;
        M.R[e] = (r <= k) ? dr * M.Rdom[e] : 0.0;
        if (k == 0) M.dsign[r] = dr;
    }
}

template <int NS>
static hipError_t launch_tree_b_ns(const BMat *mats, const int *list, int cnt, int64_t gx, int level, hipStream_t st) {
    const size_t sh = sizeof(TreeSmem<NS>);
    hipError_t e = hipFuncSetAttribute((const void *)k_tree_b<NS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    ProfScope ps("batch_tree_factor", st);
    hipLaunchKernelGGL(k_tree_b<NS>, dim3((unsigned)gx, (unsigned)cnt), dim3(64 * NS), sh, st, mats, list,
                       level);
    return hipGetLastError();
}

hipError_t launch_tree_b(const BMat *mats, const int *list, int cnt, int64_t gx, int ns, int level, hipStream_t st) {
    if (cnt <= 0 || gx <= 0) return hipSuccess;
    switch (ns) {
        case 1: return launch_tree_b_ns<1>(mats, list, cnt, gx, level, st);
        case 2: return launch_tree_b_ns<2>(mats, list, cnt, gx, level, st);
        default: return launch_tree_b_ns<4>(mats, list, cnt, gx, level, st);
    }
}

hipError_t launch_tree_t_b(const BMat *mats, const int *list, int cnt, int64_t maxP, int ns, hipStream_t st) {
    if (cnt <= 0 || !tree_t_needed(maxP, ns)) return hipSuccess;
    const size_t sh = sizeof(NodeTSmem);
    hipError_t e = hipFuncSetAttribute((const void *)k_tree_t_b, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    ProfScope ps("batch_tree_t", st);
    hipLaunchKernelGGL(k_tree_t_b, dim3((unsigned)(maxP - 1), (unsigned)cnt), dim3(kNodeThreads), sh, st, mats, list);
    return hipGetLastError();
}

hipError_t launch_sign_b(const BMat *mats, const int *list, int cnt, hipStream_t st) {
    if (cnt <= 0) return hipSuccess;
    ProfScope ps("batch_sign_normalise", st);
    hipLaunchKernelGGL(k_sign_b, dim3((unsigned)cnt), dim3(256), 0, st, mats, list);
    return hipGetLastError();
}

template <int NS>
static hipError_t launch_tree_level_ns(double *Rdom, double *Tnode, const PanelArgs &pa, const TreeArgs &ta, int keep_q,
                                       hipStream_t st) {
    const size_t sh = sizeof(TreeSmem<NS>);
    hipError_t e = hipFuncSetAttribute((const void *)k_tree<NS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    ProfScope ps("tree_factor", st);
    hipLaunchKernelGGL(k_tree<NS>, dim3((unsigned)ta.chains), dim3(64 * NS), sh, st, Rdom, Tnode, pa, ta,
                       keep_q);
    return hipGetLastError();
}

hipError_t launch_tree_level(double *Rdom, double *Tnode, const PanelArgs &pa, const TreeArgs &ta,
                             int keep_q, hipStream_t st) {
    switch (pa.ns) {
        case 1: return launch_tree_level_ns<1>(Rdom, Tnode, pa, ta, keep_q, st);
        case 2: return launch_tree_level_ns<2>(Rdom, Tnode, pa, ta, keep_q, st);
        default: return launch_tree_level_ns<4>(Rdom, Tnode, pa, ta, keep_q, st);
    }
}

hipError_t launch_tree_t(const double *Rdom, double *Tnode, const PanelArgs &pa, hipStream_t st) {
    if (!tree_t_needed(pa.P, pa.ns)) return hipSuccess;
    const size_t sh = sizeof(NodeTSmem);
    hipError_t e = hipFuncSetAttribute((const void *)k_tree_t, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    ProfScope ps("tree_t", st);
    hipLaunchKernelGGL(k_tree_t, dim3((unsigned)(pa.P - 1)), dim3(kNodeThreads), sh, st, Rdom, Tnode, pa);
    return hipGetLastError();
}

hipError_t launch_sign_normalise(const double *Rroot, int n, double *Rout, int64_t ldr, int row_off,
                                 int col_off, double *dsign, hipStream_t st) {
    ProfScope ps("sign_normalise", st);
    hipLaunchKernelGGL(k_sign_normalise, dim3(16), dim3(256), 0, st, Rroot, n, Rout, ldr, row_off,
                       col_off, dsign);
    return hipGetLastError();
}

}  // namespace tsqr
