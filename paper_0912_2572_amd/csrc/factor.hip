// factor.hip -- leaf kernels of the TSQR factorization on gfx950 (the tree
// kernels are in tree.hip).
//
// Leaf (Sec. 2.3, "the factorization of a domain is the operation performed
// on the leaves"): one 256-thread workgroup per domain.  The domain is
// streamed from HBM in chunks that live in registers; the domain's triangle
// R lives in LDS.  The first chunk gets a plain Householder QR (its top n
// rows become R); every later chunk C gets the structured QR of [R; C] --
// the paper's flat tree (Sec. 2.3) applied inside the domain, so A is read
// exactly once.  Each chunk leaves its reflectors V in place of the chunk
// and its compact-WY factor T (Sec. 2.2: H_1...H_n = I - V T V^T).
//
// The QR of a chunk is panel_qr.h's: 16-column panels whose column steps
// touch one register slot, and matrix-core updates of the other slots.
// What bounds the kernel: the column steps' latency (64 of ~900 cycles per
// 256-row chunk, one workgroup per CU when there are as many domains as CUs)
// and then the matrix cores' 312 FP64 products per wave and chunk (20,000
// cycles of ~115,000).  Leaf of 1,048,576 x 64 in 256 domains: 0.79 ms, 1.53
// TB/s of A, V and T (1.49 ms with column steps over all 64 columns); x 32:
// 0.30 (0.69); x 16: 0.09 (0.26).
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

namespace {

constexpr int kLeafWaves = 4;
constexpr int kLeafThreads = 64 * kLeafWaves;

typedef double dv2 __attribute__((ext_vector_type(2)));

// Tiles per wave and slot: chunk_rows(ns) rows over four waves.
template <int NS>
constexpr int kLeafTiles = chunk_rows(NS) / (16 * kLeafWaves);

template <int NS>
using LeafSmem = PanelSmem<kLeafWaves, NS, kLeafTiles<NS>>;

template <typename T>
__device__ __forceinline__ bool rows_aligned(const T *p, int64_t ld) {
    return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && (ld * (int64_t)sizeof(T)) % 16 == 0;
}

// A lane's place in a chunk: column cg of a slot, first row of its first row
// pair.
struct LaneAt {
    int cg, row;
};
__device__ __forceinline__ LaneAt lane_at() {
    const int lane = threadIdx.x & 63;
    return LaneAt{lane & 15, 16 * wave_index<kLeafWaves>() + 2 * (lane >> 4)};
}
// Row offset of row pair h (registers 2 h, 2 h + 1) of tile a from there.
__device__ constexpr int pair_off(int a, int h) { return 16 * kLeafWaves * a + 8 * h; }

// Rows [0, valid) x columns [0, n) of a chunk at src (ld) into c, zeros
// elsewhere (a partial chunk).  A row past `valid` reads row 0.
template <int NS, int NT>
__device__ __forceinline__ void load_chunk(d4 (&c)[NS][NT], const double *__restrict__ src, int64_t ld,
                                           int64_t valid, int n) {
    LaneAt la = lane_at();
    asm volatile("" : "+v"(la.cg), "+v"(la.row));   // nothing of this is kept across the chunks
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        const int k = la.cg + 16 * t;
        const double *p = src + (int64_t)(k < n ? k : 0) * ld;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = la.row + pair_off(a, r >> 1) + (r & 1);
                c[t][a][r] = p[row < valid ? row : 0];
            }
    }
    // (every load issued first)
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = la.cg + 16 * t < n && la.row + pair_off(a, r >> 1) + (r & 1) < valid;
                c[t][a][r] = in ? c[t][a][r] : 0.0;
            }
}

// What the lanes of a column past n read instead of the matrix.  (Pointers
// that may be either say that they point to global memory: a load through a
// generic pointer would count as an LDS access too, and every LDS wait of
// the column steps would wait for it.)
__device__ const double kZeros[512] = {};
typedef const double __attribute__((address_space(1))) *gptr;

// Loads of row pairs I0 .. I1 - 1 (of 2 NT) of a slot of a full chunk, p the
// lane's place in it (column_or_zeros), with no branch around them and
// nothing to do once the data is there, so that they stay in flight across
// the current work.  VEC: 16-byte pieces (rows_aligned must hold).
template <int NT, bool VEC, int I0, int I1>
__device__ __forceinline__ void issue_pairs(d4 (&c)[NT], gptr p) {
#pragma unroll
    for (int i = I0; i < I1; ++i) {
        const int a = i >> 1, h = i & 1;
        const gptr q = p + pair_off(a, h);
        if constexpr (VEC) {
            const dv2 v = *reinterpret_cast<const dv2 __attribute__((address_space(1))) *>(q);
            c[a][2 * h] = v.x;
            c[a][2 * h + 1] = v.y;
        } else {
            c[a][2 * h] = q[0];
            c[a][2 * h + 1] = q[1];
        }
    }
}
// A use of c: its loads are waited for here.
__device__ __forceinline__ void touch(const d4 &c) {
    const double c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
    asm volatile("" ::"v"(c0), "v"(c1), "v"(c2), "v"(c3));
}

// The lane's place in slot t of the chunk whose slot 0 is at p (kZeros for a
// column past n, or if there is no such chunk).
template <int NT>
__device__ __forceinline__ gptr column_or_zeros(const double *p, int64_t ld, int n, int t, bool live,
                                                const LaneAt la) {
    static_assert(16 * kLeafWaves * NT <= 512, "zeros for a whole column");
    const gptr col = (gptr)(p + (int64_t)(16 * t) * ld), zero = (gptr)(kZeros + la.row);
    return (live && la.cg + 16 * t < n) ? col : zero;
}

// Whether a chunk's reflectors can be stored in row pairs.
template <int NS, typename VT>
__device__ __forceinline__ bool pairs_ok(const VT *dst, int64_t ld, int64_t valid) {
    return valid >= chunk_rows(NS) && (reinterpret_cast<uintptr_t>(dst) % (2 * sizeof(VT))) == 0 && (ld % 2) == 0;
}

// Row pairs I0 .. I1 - 1 of reflector columns 16 p .. 16 p + 15 of a chunk to
// memory, dst the lane's place in the chunk's first 16 columns.  FIRST: zeros on and above the diagonal (the
// unit diagonal is implicit in memory).
template <int NT, bool FIRST, int I0, int I1, typename VT>
__device__ __forceinline__ void store_pairs(const d4 (&c)[NT], VT *__restrict__ dst, int64_t ld, int n, int p,
                                            const LaneAt la) {
    typedef VT vt2 __attribute__((ext_vector_type(2)));
    const int k = 16 * p + la.cg;
    VT *q = dst + (int64_t)(16 * p) * ld;
    if (k < n) {
#pragma unroll
        for (int i = I0; i < I1; ++i) {
            const int a = i >> 1, h = i & 1;
            double v0 = c[a][2 * h], v1 = c[a][2 * h + 1];
            if constexpr (FIRST) {
                const int row = la.row + pair_off(a, h);
                v0 = row <= k ? 0.0 : v0;
                v1 = row + 1 <= k ? 0.0 : v1;
            }
            vt2 v;
            v.x = VT(v0);
            v.y = VT(v1);
            *reinterpret_cast<vt2 *>(q + pair_off(a, h)) = v;
        }
    }
}

// The same element by element (a partial chunk, or columns that do not
// start on a pair).
template <int NT, bool FIRST, typename VT>
__device__ __forceinline__ void store_elements(const d4 (&c)[NT], VT *__restrict__ dst, int64_t ld, int64_t valid,
                                               int n, int p) {
    LaneAt la = lane_at();
    asm volatile("" : "+v"(la.cg), "+v"(la.row));   // nothing of this is kept across the chunks
    const int k = 16 * p + la.cg;
    VT *q = dst + (int64_t)k * ld + la.row;
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int off = pair_off(a, r >> 1) + (r & 1), row = la.row + off;
            const double v = (FIRST && row <= k) ? 0.0 : c[a][r];
            if (k < n && row < valid) q[off] = VT(v);
        }
}

// Columns 16 p .. 16 p + 15 of the upper triangle of an LDS matrix (row-major,
// stride ld) -> column-major n x n with zeros below the diagonal.
template <int NS>
__device__ __forceinline__ void store_upper(const double *lds, int ld, double *__restrict__ dst, int n, int p) {
    constexpr int C = 16 * NS, S = kLeafThreads / C;   // rows a pass covers, columns a pass
    const int tid = local_tid(), r = tid % C, k0 = 16 * p + tid / C;
    double v[16 / S];
#pragma unroll
    for (int u = 0; u < 16 / S; ++u) v[u] = lds[r * ld + k0 + S * u];
    double *q = dst + r + k0 * n;
#pragma unroll
    for (int u = 0; u < 16 / S; ++u) {
        const int k = k0 + S * u;
        if (r < n && k < n) q[S * u * n] = (r <= k) ? v[u] : 0.0;
    }
}

// Leaf QR of domain `dom` (step 2): the chunks of the domain in order, a
// geqrt of the first and a tpqrt of [R; chunk] for each later one.
// VT: element type of the stored reflectors (double, or float in the mixed
// mode, where they only feed the FP32 matrix-core applies).  VEC: the
// columns of A allow 16-byte loads (rows_aligned).
//
// Memory traffic goes out a few instructions per column step, so that it
// drains under the steps instead of stalling the waves that issue it in
// bursts: the steps of panel 0 load the chunk's slots 1 .. NS - 1 (which they
// do not touch) and slot 0 of the next chunk (into registers of its own),
// and the steps of a later panel store the reflectors of the panel before.
// A domain's last chunk may be a partial one (the last domain's, or every
// domain's if the row block is not a whole number of chunks): it is loaded
// with masking, all of it before its steps.
template <int NS, typename VT, bool VEC>
__device__ __forceinline__ void leaf_domain(LeafSmem<NS> &sm, const double *__restrict__ A, int64_t lda,
                                            VT *__restrict__ V, int64_t ldv, double *__restrict__ Tc,
                                            double *__restrict__ Rdom, const PanelArgs &pa, bool want_t,
                                            int64_t dom) {
    constexpr int ROWS = chunk_rows(NS), NT = kLeafTiles<NS>, LD = LeafSmem<NS>::kLd;
    const int64_t row0 = dom_row0(pa, dom);
    const int64_t nrows = dom_rows(pa, dom);
    const int64_t nfull = nrows / ROWS;          // full chunks
    const int64_t tail = nrows - nfull * ROWS;   // rows of a partial last chunk
    const int n = pa.n;
    const int64_t nn = (int64_t)n * n;
    for (int e = threadIdx.x; e < 16 * NS * LD; e += kLeafThreads) {
        sm.R[e] = 0.0;
        sm.T[e] = 0.0;
    }
    __syncthreads();
    const LaneAt la = lane_at();
    const double *pA = A + row0 + (int64_t)la.cg * lda + la.row;   // the lane's place in the chunk
    VT *pV = V + row0 + (int64_t)la.cg * ldv + la.row;
    d4 c[NS][NT], nx[NT];
    double *tc = Tc + dom_chunk0(pa, dom) * nn;
    // chunk ch: the first one, a later full one, or a partial last one
    enum { kFirst, kFull, kPartial };
    auto chunk = [&](int64_t ch, auto kind) {
        constexpr int KIND = decltype(kind)::value;
        constexpr bool FIRST = KIND == kFirst;
        constexpr int PAIRS = 2 * NT;
        const int64_t r0 = row0 + ch * ROWS, valid = ch < nfull ? (int64_t)ROWS : tail;
        const bool more = ch + 1 < nfull, pairs = want_t && pairs_ok<NS>(V + r0, ldv, valid);
        // steps 0 .. 7: the other slots, then the next chunk's slot 0
        auto load = [&](auto step) {
            constexpr int Q = decltype(step)::value;
            if constexpr (NS > 1 && Q < 4) {
#pragma unroll
                for (int t = 1; t < NS; ++t)
                    issue_pairs<NT, VEC, Q * PAIRS / 4, (Q + 1) * PAIRS / 4>(
                        c[t], column_or_zeros<NT>(pA, lda, n, t, true, la));
            } else if constexpr (Q < 8) {
                constexpr int F = NS > 1 ? 4 : 0;   // first step that loads nx
                issue_pairs<NT, VEC, (Q - F) * PAIRS / (8 - F), (Q - F + 1) * PAIRS / (8 - F)>(
                    nx, column_or_zeros<NT>(pA + ROWS, lda, n, 0, more, la));
            }
        };
        int stored = 0;   // panels whose reflectors are stored
        auto store = [&](auto step) {
            constexpr int Q = decltype(step)::value;
            if constexpr (Q < 8) {
                if (pairs)
                    store_pairs<NT, false, Q * PAIRS / 8, (Q + 1) * PAIRS / 8>(c[NS - 1], pV, ldv, n, stored, la);
            }
        };
        auto done = [&](int p, const d4 (&v)[NT], const double (&)[16]) {
            // the next chunk's slot 0 has arrived before the last stores are
            // issued: waiting for it later would wait for them too
            if constexpr (KIND == kFull && NS > 1) {
#pragma unroll
                for (int a = 0; a < NT; ++a) touch(nx[a]);
            }
            if (KIND != kFull || 16 * (p + 1) >= n) {
                if (pairs) store_pairs<NT, FIRST, 0, PAIRS>(v, pV, ldv, n, p, la);
            }
            if (want_t && !pairs) store_elements<NT, FIRST>(v, V + r0, ldv, valid, n, p);
            stored = p;
        };
        auto t_block = [&](int p) { store_upper<NS>(sm.T, LD, tc, n, p); };
        auto none = [](auto) {};
        if constexpr (KIND != kFull) {
            if constexpr (FIRST) issue_pairs<NT, VEC, 0, PAIRS>(nx, column_or_zeros<NT>(pA + ROWS, lda, n, 0, more, la));
            panel_qr<kLeafWaves, NS, NT, FIRST, false>(c, n, sm, want_t, none, none, done, t_block);
        } else {
            panel_qr<kLeafWaves, NS, NT, false, true>(c, n, sm, want_t, load, store, done, t_block);
        }
        pA += ROWS;
        pV += ROWS;
        tc += nn;
    };
    if (nfull == 0) {
        load_chunk<NS, NT>(c, A + row0, lda, tail, n);
    } else {
#pragma unroll
        for (int t = 0; t < NS; ++t)
            issue_pairs<NT, VEC, 0, 2 * NT>(c[t], column_or_zeros<NT>(pA, lda, n, t, true, la));
    }
    chunk(0, std::integral_constant<int, kFirst>{});
    for (int64_t ch = 1; ch < nfull; ++ch) {
#pragma unroll
        for (int a = 0; a < NT; ++a) c[0][a] = nx[a];
        chunk(ch, std::integral_constant<int, kFull>{});
    }
    if (nfull > 0 && tail > 0) {
        load_chunk<NS, NT>(c, A + row0 + nfull * ROWS, lda, tail, n);
        chunk(nfull, std::integral_constant<int, kPartial>{});
    }
    __syncthreads();
    for (int p = 0; 16 * p < n; ++p) store_upper<NS>(sm.R, LD, Rdom + dom * nn, n, p);
}

// Narrow panels (NS <= 2) fit two workgroups per CU (registers and LDS),
// which hides step latency whenever there are more domains than CUs.
template <int NS>
constexpr int leaf_min_blocks() { return NS <= 2 ? 2 : 1; }

}  // namespace

template <int NS, typename VT, bool VEC>
__global__ __launch_bounds__(kLeafThreads, leaf_min_blocks<NS>()) void k_leaf(const double *__restrict__ A, int64_t lda,
                                                 VT *__restrict__ V, int64_t ldv,
                                                 double *__restrict__ Tc, double *__restrict__ Rdom,
                                                 PanelArgs pa, int keep_q) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    LeafSmem<NS> &sm = *reinterpret_cast<LeafSmem<NS> *>(smem_raw);
    leaf_domain<NS, VT, VEC>(sm, A, lda, V, ldv, Tc, Rdom, pa, keep_q != 0, blockIdx.x);
}

// ---- batched forms: grid.y walks the matrix list, grid.x the domains /
// chains of the listed matrix (a workgroup past its matrix's count returns).
template <int NS>
__global__ __launch_bounds__(kLeafThreads, leaf_min_blocks<NS>()) void k_leaf_b(const BMat *__restrict__ mats,
                                                   const int *__restrict__ list) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    LeafSmem<NS> &sm = *reinterpret_cast<LeafSmem<NS> *>(smem_raw);
    const BMat &M = mats[list[blockIdx.y]];
    const int64_t dom = blockIdx.x;
    if (dom >= M.pa.P) return;
    const bool vec = rows_aligned(M.A, M.lda) && (M.pa.mb % 2) == 0;
    if (M.prec) {
        if (vec) leaf_domain<NS, float, true>(sm, M.A, M.lda, M.V32, M.pa.m, M.Tc, M.Rdom, M.pa, true, dom);
        else leaf_domain<NS, float, false>(sm, M.A, M.lda, M.V32, M.pa.m, M.Tc, M.Rdom, M.pa, true, dom);
    } else {
        if (vec) leaf_domain<NS, double, true>(sm, M.A, M.lda, M.V, M.pa.m, M.Tc, M.Rdom, M.pa, true, dom);
        else leaf_domain<NS, double, false>(sm, M.A, M.lda, M.V, M.pa.m, M.Tc, M.Rdom, M.pa, true, dom);
    }
}

template <int NS>
static hipError_t launch_leaf_b_ns(const BMat *mats, const int *list, int cnt, int64_t gx, hipStream_t st) {
    const size_t sh = sizeof(LeafSmem<NS>);
    hipError_t e = hipFuncSetAttribute((const void *)k_leaf_b<NS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    ProfScope ps("batch_leaf_factor", st);
    hipLaunchKernelGGL(k_leaf_b<NS>, dim3((unsigned)gx, (unsigned)cnt), dim3(kLeafThreads), sh, st, mats,
                       list);
    return hipGetLastError();
}

hipError_t launch_leaf_b(const BMat *mats, const int *list, int cnt, int64_t gx, int ns, hipStream_t st) {
    if (cnt <= 0 || gx <= 0) return hipSuccess;
    switch (ns) {
        case 1: return launch_leaf_b_ns<1>(mats, list, cnt, gx, st);
        case 2: return launch_leaf_b_ns<2>(mats, list, cnt, gx, st);
        default: return launch_leaf_b_ns<4>(mats, list, cnt, gx, st);
    }
}

template <int NS, typename VT, bool VEC>
static hipError_t launch_leaf_nsv(const double *A, int64_t lda, VT *V, int64_t ldv, double *Tc,
                                  double *Rdom, const PanelArgs &pa, int keep_q, const char *tag,
                                  hipStream_t st) {
    const size_t sh = sizeof(LeafSmem<NS>);
    hipError_t e = hipFuncSetAttribute((const void *)k_leaf<NS, VT, VEC>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    ProfScope ps(tag, st);
    hipLaunchKernelGGL((k_leaf<NS, VT, VEC>), dim3((unsigned)pa.P), dim3(kLeafThreads), sh, st, A, lda, V,
                       ldv, Tc, Rdom, pa, keep_q);
    return hipGetLastError();
}

template <int NS, typename VT>
static hipError_t launch_leaf_ns(const double *A, int64_t lda, VT *V, int64_t ldv, double *Tc,
                                 double *Rdom, const PanelArgs &pa, int keep_q, const char *tag,
                                 hipStream_t st) {
    // 16-byte loads need every chunk's first row 16-byte aligned: A itself,
    // every column start (lda) and every domain start (mb) must be even
    const bool vec = (reinterpret_cast<uintptr_t>(A) & 15) == 0 && (lda * (int64_t)sizeof(double)) % 16 == 0 &&
                     (pa.mb % 2) == 0;
    return vec ? launch_leaf_nsv<NS, VT, true>(A, lda, V, ldv, Tc, Rdom, pa, keep_q, tag, st)
               : launch_leaf_nsv<NS, VT, false>(A, lda, V, ldv, Tc, Rdom, pa, keep_q, tag, st);
}

template <typename VT>
static hipError_t launch_leaf_t(const double *A, int64_t lda, VT *V, int64_t ldv, double *Tc, double *Rdom,
                                const PanelArgs &pa, int keep_q, const char *tag, hipStream_t st) {
    switch (pa.ns) {
        case 1: return launch_leaf_ns<1, VT>(A, lda, V, ldv, Tc, Rdom, pa, keep_q, tag, st);
        case 2: return launch_leaf_ns<2, VT>(A, lda, V, ldv, Tc, Rdom, pa, keep_q, tag, st);
        default: return launch_leaf_ns<4, VT>(A, lda, V, ldv, Tc, Rdom, pa, keep_q, tag, st);
    }
}

hipError_t launch_leaf(const double *A, int64_t lda, double *V, int64_t ldv, double *Tc, double *Rdom,
                       const PanelArgs &pa, int keep_q, hipStream_t st) {
    return launch_leaf_t<double>(A, lda, V, ldv, Tc, Rdom, pa, keep_q, "leaf_factor", st);
}

hipError_t launch_leaf32(const double *A, int64_t lda, float *V, int64_t ldv, double *Tc, double *Rdom,
                         const PanelArgs &pa, int keep_q, hipStream_t st) {
    return launch_leaf_t<float>(A, lda, V, ldv, Tc, Rdom, pa, keep_q, "leaf_factor_v32", st);
}

}  // namespace tsqr
