// formq.hip -- the thin Q of a single-panel TSQR (n <= 64) on matrix cores.
//
// Q_1 D = Q_full [D; 0] (Sec. 2.2 uniqueness, sign matrix D).  The tree is
// applied top-down first (Sec. 2.3: the reduction tree is reused for Q):
// the root block is S_0 = D, and a node (l, r) with reflector block
// [I; U] and factor T maps its parent block S_l to
//     S_r = -U T S_l,    S_l <- S_l - T S_l.
// Each domain then expands its n x n block S_i through its chunks, last
// chunk first.  A chunk k >= 1 with reflectors [I; V_k] and factor T_k
// turns the running block X (the domain's top rows) into
//     rows of chunk k = -V_k (T_k X),   X <- X - T_k X,
// and the first chunk (unit lower trapezoidal V_0) gives
//     rows of chunk 0 = [X; 0] - V_0 T_0 (V_0top^T X).
// The chunk products run as FP64 MFMA tiles in the transposed form
// Q^T-tile = Z^T V^T, so that every store writes 16 consecutive rows of a
// column of the column-major Q.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

// n x n blocks on eight waves, n <= 16 NT: wave w owns row tile w % 4 and the
// column tiles of half w / 4 of every product.  Blocks that are multiplied sit
// in LDS (rows at form_place), a wave's own tiles of a running block in
// registers as well; the left factors (T, U) come from memory straight into
// the operand layout, 16 rows of a column to a cache line.
template <int NT>
struct FormSmem {
    double X[2][16 * NT][16 * NT];
    double Z[2][16 * NT][16 * NT];
};
// Place of column c in row r: odd rows have the halves of a 32-column span
// exchanged, so that the two rows a half wave reads fall into different banks.
template <int NT>
__device__ __forceinline__ int form_place(int r, int c) {
    return NT > 1 && 16 * NT % 32 == 0 ? c ^ ((r & 1) << 4) : c;
}

template <int NT>
struct FormTiles {
    static constexpr int JH = (NT + 1) / 2;
    using Block = double[16 * NT][16 * NT];
    int I, J0, l16, l4, n;
    bool own;
    __device__ __forceinline__ FormTiles(int n_) {
        const int w = wave_index<8>(), lane = threadIdx.x & 63;
        I = w & 3;
        J0 = (w >> 2) * JH;
        l16 = lane & 15;
        l4 = lane >> 4;
        n = n_;
        own = I < NT;
    }
    // entry kb of this lane's operand of an upper triangle: (16 I + l16, 4 kb + l4)
    __device__ __forceinline__ bool upper(int kb) const {
        const int r = 16 * I + l16, c = 4 * kb + l4;
        return r <= c && c < n;
    }
    __device__ __forceinline__ void fetch_upper(double (&a)[4 * NT], const double *__restrict__ T) const {
#pragma unroll
        for (int kb = 0; kb < 4 * NT; ++kb) a[kb] = T[upper(kb) ? 16 * I + l16 + (4 * kb + l4) * n : 0];
    }
    // this wave's tiles of an n x n block in memory (column-major, ld n)
    __device__ __forceinline__ void fetch(d4 (&x)[JH], const double *__restrict__ S) const {
#pragma unroll
        for (int j = 0; j < JH; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * I + 4 * r + l4, col = 16 * (J0 + j) + l16;
                const bool ok = row < n && col < n;
                const double s = S[ok ? row + col * n : 0];
                x[j][r] = ok ? s : 0.0;
            }
    }
    __device__ __forceinline__ void store(double *__restrict__ S, const d4 (&x)[JH]) const {
#pragma unroll
        for (int j = 0; j < JH; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * I + 4 * r + l4, col = 16 * (J0 + j) + l16;
                if (row < n && col < n) S[row + col * n] = x[j][r];
            }
    }
    __device__ __forceinline__ void put(Block &M, const d4 (&x)[JH]) const {
#pragma unroll
        for (int j = 0; j < JH; ++j)
            if (J0 + j < NT) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * I + 4 * r + l4;
                    M[row][form_place<NT>(row, 16 * (J0 + j) + l16)] = x[j][r];
                }
            }
    }
    // sum over kb of the operand (where ok(kb), else zero) times M's rows (no
    // branch: a triangle's zero tiles are multiplied)
    template <typename Ok>
    __device__ __forceinline__ void product(const double (&a)[4 * NT], const Block &M, d4 (&z)[JH], Ok ok) const {
#pragma unroll
        for (int j = 0; j < JH; ++j) z[j] = d4_zero();
#pragma unroll
        for (int kb = 0; kb < 4 * NT; ++kb) {
            const double t = ok(kb) ? a[kb] : 0.0;
#pragma unroll
            for (int j = 0; j < JH; ++j) {
                const int J = J0 + j < NT ? J0 + j : NT - 1;
                z[j] = mfma_f64(t, M[4 * kb + l4][form_place<NT>(4 * kb + l4, 16 * J + l16)], z[j]);
            }
        }
    }
    __device__ __forceinline__ void upper_product(const double (&a)[4 * NT], const Block &M, d4 (&z)[JH]) const {
        product(a, M, z, [&](int kb) { return upper(kb); });
    }
};

// Top-down tree level for the thin Q: one workgroup per chain.  Per node Z =
// T S_l, S_l <- S_l - Z, S_r = -U Z, one barrier (X and Z alternate between two
// buffers).  What bounds it: latency of the loads, then 2 x 16 k-steps of tile
// products.  Measured against four waves on padded 64 x 64 products staged
// through LDS: a level of a 256-domain tree, n = 64 36 -> 23 us (beside the
// solve), n = 16 31 -> 8 us, n = 8 20 -> 6.5 us.
template <int NT>
__global__ __launch_bounds__(512) void k_tree_down(const double *__restrict__ Rdom,
                                                   const double *__restrict__ Tnode,
                                                   double *__restrict__ S, PanelArgs pa, TreeArgs ta) {
    extern __shared__ double smem_raw[];
    FormSmem<NT> &sm = *reinterpret_cast<FormSmem<NT> *>(smem_raw);
    const FormTiles<NT> ft(pa.n);
    constexpr int JH = FormTiles<NT>::JH;
    const int64_t nn = (int64_t)pa.n * pa.n;
    const int64_t left = tree_left(ta, blockIdx.x);
    if (left >= pa.P) return;
    int64_t nr = 0;
    for (int64_t q = 1; q * ta.stride < ta.span && left + q * ta.stride < pa.P; ++q) ++nr;
    if (nr == 0) return;
    d4 x[JH];
    double t[4 * NT], u[4 * NT];
    ft.fetch(x, S + left * nn);
    ft.fetch_upper(t, Tnode + (left + nr * ta.stride) * nn);
    ft.fetch_upper(u, Rdom + (left + nr * ta.stride) * nn);
    if (ft.own) ft.put(sm.X[nr & 1], x);
    __syncthreads();
#pragma unroll 1
    for (int64_t q = nr; q >= 1; --q) {
        const int64_t right = left + q * ta.stride, next = left + (q > 1 ? q - 1 : 1) * ta.stride;
        const int cur = (int)(q & 1);
        d4 z[JH];
        if (ft.own) {
            ft.upper_product(t, sm.X[cur], z);
            ft.put(sm.Z[cur], z);
#pragma unroll
            for (int j = 0; j < JH; ++j) x[j] -= z[j];
            ft.put(sm.X[cur ^ 1], x);
        }
        ft.fetch_upper(t, Tnode + next * nn);
        __syncthreads();
        if (ft.own) {
            ft.upper_product(u, sm.Z[cur], z);
#pragma unroll
            for (int j = 0; j < JH; ++j) z[j] = -z[j];
            ft.store(S + right * nn, z);
        }
        ft.fetch_upper(u, Rdom + next * nn);
    }
    if (ft.own) ft.store(S + left * nn, x);
}

// The top levels of the top-down tree in one launch: workgroup g takes the
// domain d = g * dstride (a left of a chain at level lstop - 1), starts from
// the root block D and applies the maps of the nodes on its path down to
// level lstop (the left's S_l <- S_l - T S_l for each later right of its
// chain, then S_r = -U (T S_l) on entering a right) -- the products and
// order of k_tree_down, so the blocks are bitwise the same.  The few upper
// nodes are recomputed by each path through them; in exchange the top
// levels cost one launch and occupy only P / dstride CUs.
template <int NT>
__global__ __launch_bounds__(512) void k_tree_down_top(const double *__restrict__ Rdom,
                                                       const double *__restrict__ Tnode,
                                                       const double *__restrict__ dsign,
                                                       double *__restrict__ S, PanelArgs pa, TreePath tp,
                                                       int lstop, int64_t dstride) {
    extern __shared__ double smem_raw[];
    FormSmem<NT> &sm = *reinterpret_cast<FormSmem<NT> *>(smem_raw);
    const FormTiles<NT> ft(pa.n);
    constexpr int JH = FormTiles<NT>::JH;
    const int n = pa.n;
    const int64_t nn = (int64_t)n * n;
    const int64_t d = (int64_t)blockIdx.x * dstride;
    d4 x[JH], z[JH];
#pragma unroll
    for (int j = 0; j < JH; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * ft.I + 4 * r + ft.l4, col = 16 * (ft.J0 + j) + ft.l16;
            const double s = dsign[row < n ? row : 0];
            x[j][r] = (row == col && row < n) ? s : 0.0;
        }
    int cur = 0;
    if (ft.own) ft.put(sm.X[0], x);
    // node (left, right): the left's map, or the map into the right
    auto node = [&](int64_t right, bool enter) {
        double t[4 * NT], u[4 * NT];
        ft.fetch_upper(t, Tnode + right * nn);
        if (enter) ft.fetch_upper(u, Rdom + right * nn);
        __syncthreads();
        if (ft.own) {
            ft.upper_product(t, sm.X[cur], z);
            if (enter) {
                ft.put(sm.Z[cur], z);
            } else {
#pragma unroll
                for (int j = 0; j < JH; ++j) x[j] -= z[j];
                ft.put(sm.X[cur ^ 1], x);
            }
        }
        if (enter) {
            __syncthreads();
            if (ft.own) {
                ft.upper_product(u, sm.Z[cur], z);
#pragma unroll
                for (int j = 0; j < JH; ++j) x[j] = -z[j];
                ft.put(sm.X[cur ^ 1], x);
            }
        }
        cur ^= 1;
    };
#pragma unroll 1
    for (int L = tp.nlev - 1; L >= lstop; --L) {
        const int64_t stride = tp.stride[L], span = tp.span[L];
        const int64_t left = d / span * span;
        const int64_t qd = (d - left) / stride;
        int64_t nr = 0;
        for (int64_t q = 1; q * stride < span && left + q * stride < pa.P; ++q) ++nr;
#pragma unroll 1
        for (int64_t q = nr; q >= (qd > 1 ? qd : 1); --q) node(left + q * stride, q == qd);
    }
    if (ft.own) ft.store(S + d * nn, x);
}

// S_0 = D (n x n, column-major).
__global__ void k_seed_root(double *S, int n, const double *d) {
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
        const int r = e % n, c = e / n;
        S[e] = (r == c) ? d[r] : 0.0;
    }
}

// Expansion of a domain's block X through its chunks, last to first, n <= 16 NT
// columns: eight waves, one workgroup per domain.  Of the n x n products wave w
// owns row tile w % 4 and the column tiles of half w / 4; X and Z sit in LDS
// twice (a chunk reads one pair while the next one's are written: one barrier
// a chunk), X's own tiles in registers as well, T's operand comes from memory a
// chunk ahead.  Of the output rows wave w owns the 16-row tiles w, w + 8, ...
// of each chunk, together: an entry of Z read from LDS serves all of them, and
// the next chunk's V is read into a register as soon as the last product that
// uses it is issued.
// What bounds it: at n = 64 the matrix cores (20 thousand cycles a chunk of 256
// rows) and memory about alike, at small n memory.  Measured against four waves
// on 64 x 64 products whatever n is, V in flight within a chunk only:
// 1,048,576 x 64 (256 domains) 0.44 -> 0.32 ms, 1,048,576 x 16 0.25 -> 0.062 ms
// (4.3 TB/s), 4096 x 16 (4 domains) 0.073 -> 0.013 ms.  A branch per product (skipping T's
// zeros) or on the first chunk inside the loop cost it a wait each (0.47 ms).
template <int NT>
__global__ __launch_bounds__(512, 2) void k_form_leaf(const double *__restrict__ V, int64_t ldv,
                                                      const double *__restrict__ Tc,
                                                      const double *__restrict__ S, PanelArgs pa,
                                                      double *__restrict__ Q, int64_t ldq) {
    extern __shared__ double smem_raw[];
    FormSmem<NT> &sm = *reinterpret_cast<FormSmem<NT> *>(smem_raw);
    constexpr int NS = NT == 1 ? 1 : (NT == 2 ? 2 : 4);      // the panel's slots
    constexpr int TPW = chunk_rows(NS) / 128, JH = FormTiles<NT>::JH;
    FormTiles<NT> ft(pa.n);
    const int w = wave_index<8>(), &l16 = ft.l16, &l4 = ft.l4, I = ft.I;
    const int n = pa.n;
    const int64_t nn = (int64_t)n * n, dom = blockIdx.x, row0 = dom_row0(pa, dom), nrows = dom_rows(pa, dom);
    const int64_t nch = (nrows + pa.chunk - 1) / pa.chunk;
    const double *T0 = Tc + dom_chunk0(pa, dom) * nn;
    const bool own = ft.own;
    V += row0;
    Q += row0;

    double tk[4 * NT];   // a chunk's T
    // V of this wave's tiles in a chunk: rows past it repeat its last row,
    // columns past n column n - 1 (they meet zero rows of Z)
    double v[TPW][4 * NT];
    auto fetch_v = [&](int64_t ch, int kb) {
        const int64_t off = ch * pa.chunk;
        const int valid = (int)(nrows - off < pa.chunk ? nrows - off : pa.chunk);
        const double *p = V + off + (int64_t)(4 * kb + l4 < n ? 4 * kb + l4 : n - 1) * ldv;
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
            const int r = 16 * (w + 8 * u) + l16;
            v[u][kb] = p[r < valid ? r : valid - 1];
        }
    };
    ft.fetch_upper(tk, T0 + (nch - 1) * nn);
    d4 x[JH];
    ft.fetch(x, S + dom * nn);
#pragma unroll
    for (int kb = 0; kb < 4 * NT; ++kb) fetch_v(nch - 1, kb);
    if (own) ft.put(sm.X[(nch - 1) & 1], x);
    __syncthreads();
    auto chunk = [&](int64_t ch, auto first_) {
        constexpr bool first = decltype(first_)::value;
        const int64_t off = ch * pa.chunk;
        const int valid = (int)(nrows - off < pa.chunk ? nrows - off : pa.chunk);
        const int cur = (int)(ch & 1);
        asm volatile("" : "+v"(ft.l16), "+v"(ft.l4));   // addresses are not kept over the loop
        if constexpr (first) {
            // W = V0^T X (V0: the unit lower top of the first chunk) in the
            // free X buffer, then Z = T0 W
            double vt[4 * NT];
#pragma unroll
            for (int kb = 0; kb < 4 * NT; ++kb) {
                const int r = 4 * kb + l4, c = 16 * I + l16;
                const double t = V[(r < n && c < n) ? r + (int64_t)c * ldv : 0];
                vt[kb] = r == c ? 1.0 : t;
            }
            if (own) {
                d4 wv[JH];
                ft.product(vt, sm.X[cur], wv, [&](int kb) {
                    const int r = 4 * kb + l4, c = 16 * I + l16;
                    return r >= c && r < n;
                });
                ft.put(sm.X[cur ^ 1], wv);
            }
            __syncthreads();
        }
        if (own) {
            d4 z[JH];
            ft.upper_product(tk, sm.X[first ? cur ^ 1 : cur], z);
            ft.put(sm.Z[cur], z);
            if constexpr (!first) {
#pragma unroll
                for (int j = 0; j < JH; ++j) x[j] -= z[j];
                ft.put(sm.X[cur ^ 1], x);
            }
        }
        if constexpr (!first) ft.fetch_upper(tk, T0 + (ch - 1) * nn);
        __syncthreads();
        // Q = -V Z, plus [X; 0] on a first chunk
        if constexpr (first) {
#pragma unroll
            for (int u = 0; u < TPW; ++u) {
                const int r = 16 * (w + 8 * u) + l16;
#pragma unroll
                for (int kb = 0; kb < 4 * NT; ++kb) {
                    const int c = 4 * kb + l4;
                    v[u][kb] = r > c ? v[u][kb] : (r == c ? 1.0 : 0.0);
                }
            }
        }
        d4 acc[TPW][NT];
#pragma unroll
        for (int u = 0; u < TPW; ++u)
#pragma unroll
            for (int c = 0; c < NT; ++c) acc[u][c] = d4_zero();
#pragma unroll
        for (int kb = 0; kb < 4 * NT; ++kb) {
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const double z = sm.Z[cur][4 * kb + l4][form_place<NT>(4 * kb + l4, 16 * c + l16)];
#pragma unroll
                for (int u = 0; u < TPW; ++u) acc[u][c] = mfma_f64(z, v[u][kb], acc[u][c]);
            }
            if constexpr (!first) fetch_v(ch - 1, kb);
        }
        const bool whole = !first && valid == (int)pa.chunk && n == 16 * NT;   // no guard around the stores
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
            const int r = 16 * (w + 8 * u) + l16;
            double *q = Q + off + r + l4 * ldq;
            if (whole) {
#pragma unroll
                for (int c = 0; c < NT; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[(int64_t)(16 * c + 4 * i) * ldq] = -acc[u][c][i];
            } else if (r < valid) {
#pragma unroll
                for (int c = 0; c < NT; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int col = 16 * c + 4 * i + l4;
                        double o = -acc[u][c][i];
                        if (first && r < n) o += sm.X[cur][r][form_place<NT>(r, col)];
                        if (col < n) q[(int64_t)(16 * c + 4 * i) * ldq] = o;
                    }
            }
        }
    };
#pragma unroll 1
    for (int64_t ch = nch - 1; ch > 0; --ch) chunk(ch, std::false_type{});
    chunk(0, std::true_type{});
}

// f(std::integral_constant<int, NT>) with NT = the 16-column tiles of n.
template <typename F>
static hipError_t with_tiles(int n, F f) {
    switch ((n + 15) >> 4) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        default: return f(std::integral_constant<int, 4>{});
    }
}
static hipError_t set_smem(const void *k, size_t sh) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
}

hipError_t launch_seed_root(double *S, int n, const double *dsign, hipStream_t st) {
    ProfScope ps("seed_root", st);
    hipLaunchKernelGGL(k_seed_root, dim3(1), dim3(256), 0, st, S, n, dsign);
    return hipGetLastError();
}

hipError_t launch_tree_down_top(const double *Rdom, const double *Tnode, const double *dsign, double *S,
                                const PanelArgs &pa, const TreePath &tp, int lstop, int64_t dstride,
                                hipStream_t st) {
    return with_tiles(pa.n, [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        const size_t sh = sizeof(FormSmem<NT>);
        hipError_t e = set_smem((const void *)k_tree_down_top<NT>, sh);
        if (e != hipSuccess) return e;
        ProfScope ps("tree_down", st);
        const int64_t groups = (pa.P + dstride - 1) / dstride;
        hipLaunchKernelGGL(k_tree_down_top<NT>, dim3((unsigned)groups), dim3(512), sh, st, Rdom, Tnode, dsign, S,
                           pa, tp, lstop, dstride);
        return hipGetLastError();
    });
}

hipError_t launch_tree_down(const double *Rdom, const double *Tnode, double *S, const PanelArgs &pa,
                            const TreeArgs &ta, hipStream_t st) {
    return with_tiles(pa.n, [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        const size_t sh = sizeof(FormSmem<NT>);
        hipError_t e = set_smem((const void *)k_tree_down<NT>, sh);
        if (e != hipSuccess) return e;
        ProfScope ps("tree_down", st);
        hipLaunchKernelGGL(k_tree_down<NT>, dim3((unsigned)ta.chains), dim3(512), sh, st, Rdom, Tnode, S, pa, ta);
        return hipGetLastError();
    });
}

hipError_t launch_form_leaf(const double *V, int64_t ldv, const double *Tc, const double *S,
                            const PanelArgs &pa, double *Q, int64_t ldq, hipStream_t st) {
    return with_tiles(pa.n, [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        const size_t sh = sizeof(FormSmem<NT>);
        hipError_t e = set_smem((const void *)k_form_leaf<NT>, sh);
        if (e != hipSuccess) return e;
        ProfScope ps("form_leaf", st);
        hipLaunchKernelGGL(k_form_leaf<NT>, dim3((unsigned)pa.P), dim3(512), sh, st, V, ldv, Tc, S, pa, Q, ldq);
        return hipGetLastError();
    });
}

}  // namespace tsqr
