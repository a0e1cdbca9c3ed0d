// tslu.hip -- LU of a tall-skinny matrix with tournament pivoting (TSLU).
//
// The paper's conclusion carries TSQR's reduction tree over to LU (CALU's
// panel factorization).  What travels up the tree is a set of b candidate
// pivot rows instead of a triangle: a node stacks original rows of A (its
// children's candidates), runs Gaussian elimination with partial pivoting
// on the stack and keeps the b rows chosen as pivots.
//
//   k_tslu_leaf   one workgroup per domain: the domain's rows in stages of
//                 one 256-row stack each (its first 256 rows, then its b
//                 candidates on the next 256 - b rows), the flat tree of
//                 the TSQR leaf's chunks;
//   k_tslu_tree   one workgroup per chain of a tree level (the TSQR tree's
//                 shapes): the left's candidates stacked on each right's,
//                 as the leaf's stacks;
//   k_tslu_u      U and the unit lower L11 of A[ipiv, :] without pivoting;
//   k_tslu_l      l_i = a_i U^{-1} for every row: one row per thread, or, for
//                 up to 16,384 rows, 16 rows a wave (k_tslu_l16);
//   k_tslu_scatter  rows ipiv[k] of L <- row k of L11.
//
// Selection on a stack (select_stack): the stack's rows sit in LDS.  The
// columns go in panels of 16; a panel's elimination steps run on one wave
// alone, lane l with the panel entries of positions l, l + 64, ... in
// registers, so that a step (pivot search on the high words of |a| by 32-bit
// DPP maxima, the pivot row by lane reads, the update) needs no barrier and
// no LDS; the columns after the panel get it as one rank-16 update on the
// FP64 matrix cores by all four waves.  What bounds it: the chain of b steps,
// in instructions of that one wave (about 130 a step with four rows a lane,
// 900 cycles; a workgroup barrier and an LDS round trip alone would be 400).
// Measured against rows held whole by one thread each, with a barrier and the
// pivot row's trip through LDS in each step: leaf of 1,048,576 x 64 (256
// domains) 2.15 -> 0.90 ms, a tree level 90 -> 42 us (36 us in CALU's
// panels), U 65 -> 25 us.
#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

namespace {

constexpr int kStack = 256;
constexpr int kSelLd = 65;   // row stride of a stack in LDS (odd: a column is read without bank conflicts)

// A stack of 64 R rows.
template <int R>
struct SelSmem {
    double S[64 * R * kSelLd];   // the stack: entries still to eliminate, multipliers left of them
    double U[16 * kSelLd];       // the panel's rows of U past the panel
    int32_t gidx[64 * R];
    int32_t sel[64];
};

// Largest of the wave's 32-bit keys (in a scalar register): maxima over each
// 16-lane row by DPP shifts, then over the rows by row broadcasts, into lane
// 63, read back as a scalar.  Lanes outside a shift take the identity 0.
__device__ __forceinline__ uint32_t wave_umax(uint32_t k) {
    k = max(k, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k, 0x111, 0xf, 0xf, true));   // row_shr:1
    k = max(k, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k, 0x112, 0xf, 0xf, true));   // row_shr:2
    k = max(k, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k, 0x114, 0xf, 0xf, true));   // row_shr:4
    k = max(k, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k, 0x118, 0xf, 0xf, true));   // row_shr:8
    k = max(k, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k, 0x142, 0xa, 0xf, false));  // row_bcast:15
    k = max(k, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)k, 63);
}

// max(|a|, |b|), a NaN giving way to a number.
__device__ __forceinline__ double max_abs(double a, double b) {
    double c;
    asm("v_max_f64 %0, |%1|, |%2|" : "=v"(c) : "v"(a), "v"(b));
    return c;
}

// The pivot's place, U being the first row register whose mask is not empty:
// takes the pivot row's panel entries J .. 15 into scalars, kills its entry J.
template <int J, int U, int R>
__device__ __forceinline__ int take_row(double (&row)[16], double (&m)[R][16], const uint64_t (&mask)[R]) {
    if constexpr (U + 1 < R) {
        if (!mask[U]) return take_row<J, U + 1, R>(row, m, mask);
    }
    const int src = __builtin_ctzll(mask[U]);
#pragma unroll
    for (int j = J; j < 16; ++j) row[j] = wave_bcast(m[U][j], src);
    if ((int)(threadIdx.x & 63) == src) m[U][J] = __builtin_nan("");
    return src + 64 * U;
}

// Step Q of partial-pivoting elimination on panel p, on one wave (row r of
// lane l: stack position l + 64 r, its panel entries in m[r]).  The pivot is
// the live row of largest |m[Q]| (a NaN ranks below every number, ties go to
// the lower stack position); every other live row takes l = m[Q] * (1 /
// pivot) (one reciprocal: the multipliers only steer the selection; U and L
// are computed from the chosen rows afterwards), kept in m[Q], and updates
// its entries past Q; a zero pivot eliminates nothing.  A chosen row's entries
// from Q on are NaN: they lose every search and need no test in the update
// (nothing reads them again); `dead` (bit r) tells such a row from a live one
// only where no number is left.
template <int R, int Q>
struct SelStep {
    __device__ __forceinline__ static void run(int32_t *sel, double (&m)[R][16], uint32_t &dead, int nq) {
        if (Q < nq) {
            const int lane = threadIdx.x & 63;
            double top = max_abs(m[0][Q], 0.0);
#pragma unroll
            for (int r = 1; r < R; ++r) top = max_abs(top, m[r][Q]);
            // the largest high word first: where one lane has it, that lane's value
            const uint32_t hi = (uint32_t)__double2hiint(top), lo = (uint32_t)__double2loint(top);
            const uint32_t hmax = wave_umax(hi);
            const uint64_t have = __ballot(hi == hmax);
            uint32_t lmax = (uint32_t)__builtin_amdgcn_readlane((int)lo, __builtin_ctzll(have));
            if (have & (have - 1)) lmax = wave_umax(hi == hmax ? lo : 0u);
            const double best = __hiloint2double((int)hmax, (int)lmax);
            uint64_t mask[R], any = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) any |= mask[r] = __ballot(fabs(m[r][Q]) == best);
            if (!any) {
#pragma unroll
                for (int r = 0; r < R; ++r) mask[r] = __ballot(!(dead >> r & 1u));
            }
            double row[16];
            const int at = take_row<Q, 0, R>(row, m, mask);
            if (lane == 0) sel[Q] = at;
            dead |= (lane == (at & 63)) ? 1u << (at >> 6) : 0u;
            const double rv = (row[Q] != 0.0) ? 1.0 / row[Q] : 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                m[r][Q] *= rv;
#pragma unroll
                for (int j = Q + 1; j < 16; ++j) m[r][j] = fma(-m[r][Q], row[j], m[r][j]);
            }
        }
        if constexpr (Q + 1 < 16) SelStep<R, Q + 1>::run(sel, m, dead, nq);
    }
};

// U rows of a panel for column slot s: u = L11^{-1} S[row(k)][slot s], rows
// row(k), k = 0..15, of the stack S in pivot order (row_at: lane k's row).
__device__ __forceinline__ void panel_u(const double *S, int row_at, int p, int s, double (&u)[16]) {
    const int cg = threadIdx.x & 15;
    double nl[16];
    // lane cg: its pivot row's multipliers (left of the diagonal)
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const double v = S[row_at * kSelLd + 16 * p + k];
        nl[k] = k < cg ? -v : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int row = __builtin_amdgcn_readlane(row_at, k);
        u[k] = S[row * kSelLd + 16 * s + cg];
    }
    lower_solve<0>(u, nl, [](double v, int) { return v; });
}

// C -= L U for NT 16-row tiles of a stack (S: their first row), panel p, slots
// s0 .. s1 - 1; U: 16 rows of stride kSelLd.
template <int NT>
__device__ __forceinline__ void rank16_update(double *S, const double *U, int p, int s0, int s1) {
    const int lane = threadIdx.x & 63, cg = lane & 15, rg = lane >> 4;
    double av[NT][4];
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) av[a][r] = -S[(16 * a + cg) * kSelLd + 16 * p + 4 * r + rg];
    for (int s = s0; s < s1; ++s) {
        double bv[4];
        d4 c[NT];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) bv[kb] = U[(4 * kb + rg) * kSelLd + 16 * s + cg];
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) c[a][r] = S[(16 * a + 4 * r + rg) * kSelLd + 16 * s + cg];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int a = 0; a < NT; ++a) c[a] = mfma_f64(av[a][kb], bv[kb], c[a]);
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[(16 * a + 4 * r + rg) * kSelLd + 16 * s + cg] = c[a][r];
    }
}

// A row's b entries into its LDS row (zeros past b), in batches of 32 loads.
__device__ __forceinline__ void fetch_row(double (&v)[64], const double *__restrict__ src, int64_t lda, int b) {
#pragma unroll
    for (int k = 0; k < 64; ++k) v[k] = src[(int64_t)(k < b ? k : 0) * lda];
}
__device__ __forceinline__ void put_row(double *S, const double (&v)[64], int b, bool live) {
#pragma unroll
    for (int k = 0; k < 64; ++k) S[k] = (live && k < b) ? v[k] : 0.0;
}

// The stack in sm.S (64 R rows, `rows` of them live; their rows of A in
// sm.gidx) on four waves: the kb = min(b, rows) selection steps, then
// gidx[0 .. kb-1] <- the chosen rows in pivot order.  Returns kb.
template <int R>
__device__ __forceinline__ int select_stack(SelSmem<R> &sm, int rows, int b) {
    const int t = threadIdx.x, w = wave_index<4>(), lane = t & 63, cg = lane & 15;
    const int kb = b < rows ? b : rows;
    const int np = (kb + 15) >> 4;
    uint32_t dead = 0;   // bit r: position lane + 64 r is not (or no longer) live
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (lane + 64 * r >= rows) dead |= 1u << r;
    __syncthreads();
#pragma unroll 1
    for (int p = 0; p < np; ++p) {
        if (w == 0) {
            double m[R][16];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int j = 0; j < 16; ++j)   // canonical: no signalling NaN reaches the search
                    m[r][j] = __builtin_canonicalize(sm.S[(lane + 64 * r) * kSelLd + 16 * p + j]);
#pragma unroll
            for (int r = 0; r < R; ++r) m[r][0] = (dead >> r & 1u) ? __builtin_nan("") : m[r][0];
            SelStep<R, 0>::run(sm.sel + 16 * p, m, dead, kb - 16 * p);
            if (p + 1 < np) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int j = 0; j < 16; ++j) sm.S[(lane + 64 * r) * kSelLd + 16 * p + j] = m[r][j];
            }
        }
        __syncthreads();
        if (p + 1 == np) break;
        if (w < np - p - 1) {
            const int s = p + 1 + w;
            double u[16];
            panel_u(sm.S, sm.sel[16 * p + cg], p, s, u);
            if (lane < 16) {
#pragma unroll
                for (int k = 0; k < 16; ++k) sm.U[k * kSelLd + 16 * s + cg] = u[k];
            }
        }
        __syncthreads();
        rank16_update<R>(sm.S + 16 * R * w * kSelLd, sm.U, p, p + 1, np);
        __syncthreads();
    }
    const int32_t g = (t < kb) ? sm.gidx[sm.sel[t]] : 0;
    __syncthreads();
    if (t < kb) sm.gidx[t] = g;
    return kb;
}

}  // namespace

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_tslu_leaf(const double *__restrict__ A, int64_t lda, PanelArgs pa, int b, int32_t *__restrict__ cand) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    SelSmem<4> &sm = *reinterpret_cast<SelSmem<4> *>(smem_raw);
    const int64_t dom = blockIdx.x;
    const int64_t row0 = dom_row0(pa, dom), end = row0 + dom_rows(pa, dom);
    const int t = threadIdx.x;
    // stage by stage: positions 0 .. nc - 1 the candidates so far, then `take`
    // new rows; a thread past the candidates loads its next row (whatever the
    // candidates turn out to be) while the current stack is eliminated
    int64_t pos = row0;
    int nc = 0;
    int take = (int)((end - pos < kStack) ? end - pos : kStack);
    double v[64];
    fetch_row(v, A + (t < take ? pos + t : pos), lda, b);
    while (true) {
        const int rows = nc + take;
        if (t >= nc && t < rows) sm.gidx[t] = (int32_t)(pos + (t - nc));
        __syncthreads();
        if (t < nc) fetch_row(v, A + sm.gidx[t], lda, b);
        put_row(sm.S + t * kSelLd, v, b, t < rows);
        pos += take;
        // every later stage follows min(b, rows) = b candidates
        const int room = kStack - b;
        take = (int)((end - pos < room) ? end - pos : room);
        if (take > 0) fetch_row(v, A + ((t >= b && t < b + take) ? pos + (t - b) : pos), lda, b);
        nc = select_stack<4>(sm, rows, b);
        __syncthreads();
        if (take <= 0) break;
    }
    if (t < b) cand[dom * b + t] = sm.gidx[t];
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_tslu_tree(const double *__restrict__ A, int64_t lda, PanelArgs pa, TreeArgs ta, int b,
                 int32_t *__restrict__ cand) {
    extern __shared__ __attribute__((aligned(64))) double smem_raw[];
    SelSmem<2> &sm = *reinterpret_cast<SelSmem<2> *>(smem_raw);
    const int64_t g = blockIdx.x;
    const int64_t left = (g / ta.width) * ta.span + g % ta.width;
    if (left >= pa.P) return;
    const int t = threadIdx.x, r = t & 127, h = t >> 7;   // two threads a row, 32 columns each
    for (int64_t q = 1; q * ta.stride < ta.span && left + q * ta.stride < pa.P; ++q) {
        const int64_t right = left + q * ta.stride;
        const bool live = r < 2 * b;
        const int32_t gi = live ? ((r < b) ? cand[left * b + r] : cand[right * b + (r - b)]) : 0;
        if (h == 0) sm.gidx[r] = gi;
        double v[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) v[k] = A[gi + (int64_t)(32 * h + k < b ? 32 * h + k : 0) * lda];
#pragma unroll
        for (int k = 0; k < 32; ++k) sm.S[r * kSelLd + 32 * h + k] = (live && 32 * h + k < b) ? v[k] : 0.0;
        select_stack<2>(sm, 2 * b, b);
        if (t < b) cand[left * b + t] = sm.gidx[t];
        __syncthreads();
    }
}

// Step Q of the no-pivot LU of panel p, lane i holding row i's panel entries:
// rows below row 16 p + Q divide by the pivot and update their entries past
// Q, the pivot row broadcast by lane reads; the other rows are left alone (a
// multiplier of zero would turn their entries into NaN under an infinity of
// the pivot row).  A zero pivot eliminates nothing and sets bit Q of `zeros`.
template <int Q>
struct NoPivotStep {
    __device__ __forceinline__ static void run(double (&m)[16], int i, int p, int nq, uint32_t &zeros) {
        if (Q < nq) {
            const int k = 16 * p + Q;
            double row[16];
#pragma unroll
            for (int j = Q; j < 16; ++j) row[j] = wave_bcast(m[j], k);
            const bool zero = row[Q] == 0.0;
            zeros |= zero ? 1u << Q : 0u;
            if (i > k && !zero) {
                m[Q] /= row[Q];
#pragma unroll
                for (int j = Q + 1; j < 16; ++j) m[j] = fma(-m[Q], row[j], m[j]);
            }
        }
        if constexpr (Q + 1 < 16) NoPivotStep<Q + 1>::run(m, i, p, nq, zeros);
    }
};

// U and the unit lower L11 of A[ipiv, :] by elimination without pivoting, in
// 16-column panels as in select_stack: the steps on one wave (lane i owns row
// i), the updates on four.  info: the first zero U_jj (1-based), else 0.  What
// stands below a zero U_jj goes to L11 as it is; in S zeros take its place, so
// that the later columns' updates skip it as the steps do.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_tslu_u(const double *__restrict__ A, int64_t lda, int b, const int32_t *__restrict__ cand,
              int64_t *__restrict__ ipiv, double *__restrict__ U, int64_t ldu, double *__restrict__ L11,
              int32_t *__restrict__ dinfo) {
    __shared__ double S[64 * kSelLd];
    __shared__ double Up[16 * kSelLd];
    __shared__ uint32_t skip[4];   // columns whose pivot is zero, a word per panel
    const int t = threadIdx.x, w = wave_index<4>(), i = t & 63, cg = i & 15;
    const int32_t gi = (i < b) ? cand[i] : 0;
    if (t < b) ipiv[t] = gi;
    {
        // wave w: columns w, w + 4, ...
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = A[gi + (int64_t)(w + 4 * u < b ? w + 4 * u : 0) * lda];
#pragma unroll
        for (int u = 0; u < 16; ++u) S[i * kSelLd + w + 4 * u] = (i < b && w + 4 * u < b) ? v[u] : 0.0;
    }
    __syncthreads();
    int info = 0;
    const int np = (b + 15) >> 4;
    double *row = S + i * kSelLd;
#pragma unroll 1
    for (int p = 0; p < np; ++p) {
        if (w == 0) {
            double m[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) m[j] = row[16 * p + j];
            uint32_t zeros = 0;
            NoPivotStep<0>::run(m, i, p, b - 16 * p, zeros);
            if (zeros) {
                if (!info) info = 16 * p + __builtin_ctz(zeros) + 1;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int k = 16 * p + j;
                    if (k < i && (zeros >> j & 1u)) {
                        if (i < b) L11[i + (int64_t)k * 64] = m[j];
                        m[j] = 0.0;
                    }
                }
            }
            if (i == 0) skip[p] = zeros;
#pragma unroll
            for (int j = 0; j < 16; ++j) row[16 * p + j] = m[j];
        }
        __syncthreads();
        if (p + 1 == np) break;
        if (w < np - p - 1) {
            const int s = p + 1 + w;
            double u[16];
            panel_u(S, 16 * p + cg, p, s, u);
            if (i < 16) {
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    Up[k * kSelLd + 16 * s + cg] = u[k];
                    S[(16 * p + k) * kSelLd + 16 * s + cg] = u[k];   // the panel's rows are U now
                }
            }
        }
        __syncthreads();
        // the rows below the panel take its update, a tile per wave
        if (w > p) rank16_update<1>(S + 16 * w * kSelLd, Up, p, p + 1, np);
        __syncthreads();
    }
    if (i < b) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int k = w + 4 * u;
            if (k < b) {
                const double v = row[k];
                U[i + (int64_t)k * ldu] = (i <= k) ? v : 0.0;
                if (!(k < i && (skip[k >> 4] >> (k & 15) & 1u)))
                    L11[i + (int64_t)k * 64] = (k < i) ? v : (k == i ? 1.0 : 0.0);
            }
        }
    }
    if (t == 0 && dinfo) *dinfo = info;
}

// l_i = a_i U^{-1} (l U = a_i, column by column, l_k = 0 where U_kk = 0)
// for rows i of [0, m); U in LDS, read by every lane at the same address.
__global__ __launch_bounds__(256) void k_tslu_l(const double *__restrict__ A, int64_t lda, int64_t m, int b,
                                                const double *__restrict__ U, int64_t ldu, double *__restrict__ L,
                                                int64_t ldl) {
    __shared__ double Us[64 * 64];
    {
        // every load in flight before the LDS stores
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = threadIdx.x + 256 * u, r = e & 63, c = e >> 6;
            v[u] = (r < b && c < b) ? U[r + (int64_t)c * ldu] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) Us[threadIdx.x + 256 * u] = v[u];
    }
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    double l[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) l[k] = (k < b) ? A[i + (int64_t)k * lda] : 0.0;
#pragma unroll
    for (int k = 0; k < 64; ++k) {
        if (k < b) {
            double s = l[k];
#pragma unroll
            for (int j = 0; j < k; ++j) s = fma(-l[j], Us[j + 64 * k], s);
            const double d = Us[k + 64 * k];
            l[k] = (d == 0.0) ? 0.0 : s / d;
        }
    }
#pragma unroll
    for (int k = 0; k < 64; ++k)
        if (k < b) L[i + (int64_t)k * ldl] = l[k];
}

// The same for few rows: 16 of them on one wave (solve_rows16 with L = U^T;
// past b, U is the identity).
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_tslu_l16(const double *__restrict__ A, int64_t lda, int64_t m, int b, const double *__restrict__ U,
                int64_t ldu, double *__restrict__ L, int64_t ldl) {
    __shared__ double X[16][17];
    const int lane = threadIdx.x, l16 = lane & 15, l4 = lane >> 4;
    const int64_t r = (int64_t)blockIdx.x * 16 + l16;
    const double *__restrict__ Ar = A + (r < m ? r : m - 1);
    auto u_at = [&](int i, int j) {   // i <= j
        const double v = U[j < b ? i + (int64_t)j * ldu : 0];
        return j < b ? v : (i == j ? 1.0 : 0.0);
    };
    d4 c[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = 16 * t + 4 * q + l4;
            const double v = Ar[(int64_t)(j < b ? j : 0) * lda];
            c[t][q] = j < b ? v : 0.0;
        }
    double nl[4][16], dg[4], lo[4][4][4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        dg[p] = u_at(16 * p + l16, 16 * p + l16);
#pragma unroll
        for (int i = 0; i < 16; ++i) nl[p][i] = u_at(16 * p + (i < l16 ? i : l16), 16 * p + l16);
#pragma unroll
        for (int t = p + 1; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) lo[p][t][q] = u_at(16 * p + 4 * q + l4, 16 * t + l16);
    }
    solve_rows16(
        c, nl, lo, X,
        [&](double v, int p, int K) {
            const double d = wave_bcast(dg[p], K);
            return d == 0.0 ? 0.0 : v / d;
        },
        [&](int j, double x) {
            if (r < m && j < b) L[r + (int64_t)j * ldl] = x;
        });
}

__global__ void k_tslu_scatter(const int64_t *__restrict__ ipiv, int b, const double *__restrict__ L11,
                               double *__restrict__ L, int64_t ldl) {
    for (int e = threadIdx.x; e < b * b; e += blockDim.x) {
        const int r = e % b, c = e / b;
        L[ipiv[r] + (int64_t)c * ldl] = L11[r + 64 * c];
    }
}

hipError_t launch_tslu(const double *A, int64_t lda, const PanelArgs &pa, const std::vector<TreeArgs> &levels,
                       int b, int32_t *cand, double *L11, double *L, int64_t ldl, double *U, int64_t ldu,
                       int64_t *ipiv, int32_t *dinfo, hipStream_t st) {
    hipError_t e = hipFuncSetAttribute((const void *)k_tslu_leaf, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)sizeof(SelSmem<4>));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k_tslu_tree, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)sizeof(SelSmem<2>));
    if (e != hipSuccess) return e;
    {
        ProfScope ps("tslu_leaf", st);
        hipLaunchKernelGGL(k_tslu_leaf, dim3((unsigned)pa.P), dim3(256), sizeof(SelSmem<4>), st, A, lda, pa, b, cand);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    for (const TreeArgs &ta : levels) {
        ProfScope ps("tslu_tree", st);
        hipLaunchKernelGGL(k_tslu_tree, dim3((unsigned)ta.chains), dim3(256), sizeof(SelSmem<2>), st, A, lda, pa, ta, b, cand);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    {
        ProfScope ps("tslu_u", st);
        hipLaunchKernelGGL(k_tslu_u, dim3(1), dim3(256), 0, st, A, lda, b, cand, ipiv, U, ldu, L11, dinfo);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    {
        ProfScope ps("tslu_l", st);
        // A thread per row moves more rows a second, but its chain of 2,016
        // multiply-adds takes 29 us however few the rows are.  16 rows a wave:
        // 14 us for 4,096 rows, 20 for 16,384 (a wave per SIMD), 66 for 65,536
        // (38 with a thread per row).
        if (pa.m <= 16 * 4 * kComputeUnits)
            hipLaunchKernelGGL(k_tslu_l16, dim3((unsigned)((pa.m + 15) / 16)), dim3(64), 0, st, A, lda, pa.m, b, U,
                               ldu, L, ldl);
        else
            hipLaunchKernelGGL(k_tslu_l, dim3((unsigned)((pa.m + 255) / 256)), dim3(256), 0, st, A, lda, pa.m, b, U,
                               ldu, L, ldl);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    ProfScope ps("tslu_scatter", st);
    hipLaunchKernelGGL(k_tslu_scatter, dim3(1), dim3(256), 0, st, ipiv, b, L11, L, ldl);
    return hipGetLastError();
}

}  // namespace tsqr
