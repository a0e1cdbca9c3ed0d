// apply_mfma.hip -- leaf part of Q^T B / Q B on matrix cores: a chained form
// for blocks of 16 or 32 columns of B (the trailing update between 64-column
// panels, many right-hand sides) and a three-pass form for up to 16 columns
// (least squares, refinement corrections).
//
// Per chunk of a domain (compact-WY factor I - Y T Y^T, Sec. 2.2):
//     W = Yb + V^T B_c          (Yb = the domain's top n rows; 0 on a first
//                                chunk, whose V has an implicit unit diagonal)
//     Z = T^T W  (Q^T)  or  T W  (Q)
//     Yb -= Z,   B_c -= V Z
// W is reduced over the chunk's rows by 16x16x4 MFMA tiles with the row index
// as the reduction dimension (each wave takes a quarter of the rows, the
// four partials meet in LDS).
//
// Two precisions share the code: FP64 (V in FP64, v_mfma_f64_16x16x4f64) and
// the mixed mode's FP32 path (V stored in FP32, v_mfma_f32_16x16x4f32 with
// FP32 accumulation, W and Z in FP32).  B and the running top rows Yb stay
// FP64, and B is updated as B - (V Z) with only the product in the tile
// precision, so an FP32 apply perturbs B by about u32 times the size of the
// update rather than u32 times |B|.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma.h"
#include "panel_qr.h"
#include "prof.h"

namespace tsqr {

constexpr int KBM = 16;   // most columns of B of the three-pass form

// ---------------------------------------------------------------------------
// Chained leaf apply: one workgroup per domain and block of 16 NB columns walks
// the domain's chunks.  A wave owns a quarter of each chunk's rows.  Its rows of
// V and B come from memory once, a column per load (lane = row: 512 consecutive
// bytes; the operand layouts' own order would touch a cache line per lane, and
// the address unit then bounds the kernel), the next chunk's loads in flight
// while the current chunk is processed, and pass to the matrix cores' layouts
// through the wave's own part of LDS (no barrier):
//   W:  V^T B over the wave's rows; the waves' partials meet in LDS, wave w
//       summing reflectors 16 w .. 16 w + 15 and adding its rows of Yb (in
//       registers for the whole chain);
//   Z:  op(T) W, the same rows per wave;
//   B:  B - V Z, the product summed by itself (one rounding at B's size; summed
//       into B it is one per four columns of V, and ||B - Q Q^T B|| a tenth to a
//       fifth larger), stored by columns again.
// What bounds it: per chunk of 256 rows, n = 64 and 32 columns, 16.4 thousand
// cycles of FP64 tiles on each of a compute unit's four waves, of about 30
// thousand (the rest are the LDS passes and the seven barriers of W and Z),
// with 256 KB of loads and stores.  Measured against one 16-column block per
// workgroup with both operands read from memory in their own layouts and
// nothing in flight between phases: trailing updates of 131,072 x 512 (7
// launches, 448 .. 64 columns) 5.03 -> 2.41 ms; Q^T B and Q B of 300,001 x 40,
// 24 columns, 0.54 -> 0.146 ms each; FP32 reflectors, 1,048,576 x 64 on 64
// columns, 0.58 -> 0.26 ms.

// Row of a 16-row tile of B (in load order) that row i of a product tile is.
template <typename Tile>
__device__ __forceinline__ int tile_row_of(int i) {
    if constexpr (sizeof(typename Tile::T) == 8) return 4 * (i & 3) + (i >> 2);
    else return i;
}

// Place of row r in column c of a wave's part: the 16-byte pieces of a column
// are permuted by the column (exclusive or on the low four bits), so that 16
// columns at one row, and the 16 rows of a tile in neighbouring columns, fall
// into different banks.
template <typename T>
__device__ __forceinline__ int row_place(int r, int c) {
    if constexpr (sizeof(T) == 8) return r ^ (2 * (((c & 1) << 3) | ((c >> 1) & 7)));
    else return r ^ (4 * (((c & 3) << 2) | ((c >> 2) & 3)));
}

// LOW: no domain has more than half a chunk's rows.
template <typename Tile, int NT, int NB, bool LOW>
struct LeafApplySmem {
    using T = typename Tile::T;
    static constexpr int RT = NT == 1 && !LOW ? 8 : 4;   // 16-row tiles of a wave (chunk_rows)
    T V[4][16 * NT][16 * RT];                    // [wave][reflector][row_place]
    // in turn: per wave 16 columns of B; the partials of W that cross waves,
    // W, Z; Yb's exchange
    alignas(64) unsigned char x[4 * 16 * 16 * RT * sizeof(double)];
    static_assert(sizeof(x) >= 3 * NT * 64 * sizeof(typename Tile::Acc) &&
                      sizeof(x) >= 16 * NT * 16 * NB * sizeof(double), "every use fits");
};
static_assert(sizeof(LeafApplySmem<TileF64, 4, 2, false>) <= 160 * 1024, "fits a CU's LDS");

// The work of one chain: domain `dom`, columns c0 .. c0 + kc - 1, in groups of
// 8 domains x ncb column blocks, the column blocks of one domain 8 items
// apart.  Workgroup g takes items g, g + gridDim.x, ... (a multiple of 8), and
// workgroups go to the 8 XCDs round-robin by index: a domain's column blocks
// share one XCD (one L2) and run side by side, so that its V comes from HBM
// about once instead of ncb times.
struct ApplyItem {
    int64_t dom, row0, nrows, nch, c0;
    int kc;
};
template <int NB>
__device__ __forceinline__ bool apply_item(const PanelArgs &pa, int64_t k, int ncb, int64_t g, ApplyItem &it) {
    const int64_t per = 8 * (int64_t)ncb, within = g % per;
    it.dom = (g / per) * 8 + within % 8;
    if (it.dom >= pa.P) return false;
    it.c0 = within / 8 * (16 * NB);
    it.kc = (int)((k - it.c0 < 16 * NB) ? k - it.c0 : 16 * NB);
    it.row0 = dom_row0(pa, it.dom);
    it.nrows = dom_rows(pa, it.dom);
    it.nch = (it.nrows + pa.chunk - 1) / pa.chunk;
    return true;
}

template <typename Tile, int NT, int NB, bool LOW, bool QT>
__device__ __forceinline__ void leaf_apply_chains(LeafApplySmem<Tile, NT, NB, LOW> &sm,
                                                  const typename Tile::T *__restrict__ Vp, int64_t ldv,
                                                  const double *__restrict__ Tc, const PanelArgs &pa,
                                                  const double *Bsrcp, int64_t ldbs, double *Bp, int64_t ldb,
                                                  int64_t k, int ncb) {
    using T = typename Tile::T;
    using Acc = typename Tile::Acc;
    constexpr int RT = LeafApplySmem<Tile, NT, NB, LOW>::RT, H = RT / 4;   // H rows per lane: lane, lane + 64
    // Low domains' rows are one or two waves', and one chain of sums over 64 of
    // them loses more than four over 16: the tiles' sums meet by themselves
    constexpr bool kTileSums = LOW;
    const int w = wave_index<4>();
    int lane = threadIdx.x & 63;
    const int n = pa.n;
    const bool own = w < NT;   // this wave sums reflectors 16 w ..
    T(*Vw)[16 * RT] = sm.V[w];
    double(*Bw)[16 * RT] = reinterpret_cast<double(*)[16][16 * RT]>(sm.x)[w];
    T(*Wx)[16 * NB] = reinterpret_cast<T(*)[16 * NB]>(sm.x);
    Acc(*red)[64] = reinterpret_cast<Acc(*)[64]>(sm.x);
    double(*Yx)[16 * NB] = reinterpret_cast<double(*)[16 * NB]>(sm.x);

    // Rows past a short chunk repeat its last row (and are zero in B), columns
    // past n column n - 1 (their rows of W are cleared, so that Z is zero
    // there), columns past kc column kc - 1 (not stored).
    T v[H][16 * NT];
    double bl[H][16 * NB];
    // part `i` of RT of the loads of chunk ch of an item
    auto fetch = [&](const ApplyItem &it, int64_t ch, int i) {
        const int64_t off = ch * pa.chunk;
        const int valid = (int)(it.nrows - off < pa.chunk ? it.nrows - off : pa.chunk);
        const T *Vc = Vp + it.row0 + off;
        const double *Bc = Bsrcp + it.c0 * ldbs + it.row0 + off;
        constexpr int CB = 16 * NB / 4, CV = 16 * NT / 4;
        const int h = i >> 2, i4 = i & 3;
        const int r = 16 * RT * w + 64 * h + lane, rc = r < valid ? r : valid - 1;
#pragma unroll
        for (int c = CB * i4; c < CB * (i4 + 1); ++c)
            bl[h][c] = (Bc + (int64_t)(c < it.kc ? c : it.kc - 1) * ldbs)[rc];
#pragma unroll
        for (int c = CV * i4; c < CV * (i4 + 1); ++c) v[h][c] = (Vc + (int64_t)(c < n ? c : n - 1) * ldv)[rc];
    };

    ApplyItem it, nx;
    int64_t g = blockIdx.x;
    if (!apply_item<NB>(pa, k, ncb, g, it)) return;
#pragma unroll
    for (int i = 0; i < RT; ++i) fetch(it, QT ? 0 : it.nch - 1, i);
    const int64_t items = (pa.P + 7) / 8 * 8 * ncb;
#pragma unroll 1
    for (;;) {
        // this item, and the next (a padding item has none after it)
        g += gridDim.x;
        const bool more = g < items && apply_item<NB>(pa, k, ncb, g, nx);
        const int64_t row0 = it.row0, nrows = it.nrows, nch = it.nch;
        const int kc = it.kc;
        const double *Tk0 = Tc + dom_chunk0(pa, it.dom) * (int64_t)n * n;
        const double *Bsrc = Bsrcp + it.c0 * ldbs + row0;
        double *B = Bp + it.c0 * ldb + row0;
        double y[NB][4];
        int l16 = lane & 15, l4 = lane >> 4;
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * w + Tile::drow(r, lane), c = 16 * j + l16;
                y[j][r] = 0.0;
                if constexpr (!QT) {
                    const double x = Bsrc[(row < n ? row : 0) + (int64_t)(c < kc ? c : kc - 1) * ldbs];
                    y[j][r] = row < n ? x : 0.0;
                }
            }
#pragma unroll 1
        for (int64_t s = 0; s < nch; ++s) {
            const int64_t ch = QT ? s : nch - 1 - s, off = ch * pa.chunk;
            const int valid = (int)(nrows - off < pa.chunk ? nrows - off : pa.chunk);
            const bool first = ch == 0;
            // addresses are computed where they are used, not kept over the loop
            asm volatile("" : "+v"(lane));
            l16 = lane & 15;
            l4 = lane >> 4;
            if (first) {
                if constexpr (!QT) {   // a first chunk's top rows are Yb
                    __syncthreads();
                    if (own) {
#pragma unroll
                        for (int j = 0; j < NB; ++j)
#pragma unroll
                            for (int r = 0; r < 4; ++r) Yx[16 * w + Tile::drow(r, lane)][16 * j + l16] = y[j][r];
                    }
                    __syncthreads();
                    if (w == 0) {
#pragma unroll
                        for (int c = 0; c < 16 * NB; ++c) {
                            const double x = Yx[lane < n ? lane : 0][c];
                            bl[0][c] = lane < n ? x : bl[0][c];
                        }
                    }
                    __syncthreads();
                }
                if (w == 0) {   // unit lower trapezoid
#pragma unroll
                    for (int c = 0; c < 16 * NT; ++c) v[0][c] = lane > c ? v[0][c] : (lane == c ? T(1) : T(0));
                }
            }
            if (valid < (int)pa.chunk) {
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int c = 0; c < 16 * NB; ++c) bl[h][c] = 16 * RT * w + 64 * h + lane < valid ? bl[h][c] : 0.0;
            }
            double b[RT][NB][4];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int c = 0; c < 16; ++c) Bw[c][row_place<double>(64 * h + lane, c)] = bl[h][16 * j + c];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int h = 0; h < 4; h += 2) {
                        const double2 p =
                            *reinterpret_cast<const double2 *>(&Bw[l16][row_place<double>(16 * rt + 4 * l4 + h, l16)]);
                        b[rt][j][h] = p.x;
                        b[rt][j][h + 1] = p.y;
                    }
            }
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int c = 0; c < 16 * NT; ++c) Vw[c][row_place<T>(64 * h + lane, c)] = v[h][c];
            // op(T)'s operand: entries (q, i) or (i, q), i = 16 w + l16, q = 16 t + 4 u + l4
            const double *Tk = Tk0 + ch * (int64_t)n * n;
            double tk[NT][4];
            auto t_at = [&](int t, int u, bool &ok) {
                const int i = 16 * w + l16, q = 16 * t + 4 * u + l4;
                const int r = QT ? q : i, c = QT ? i : q;
                ok = r <= c && c < n;
                return ok ? r + c * n : 0;
            };
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    bool ok;
                    tk[t][u] = Tk[t_at(t, u, ok)];
                }
            asm volatile("" : "+v"(lane));
            l16 = lane & 15;
            l4 = lane >> 4;
            // W over this wave's rows, the next chunk's loads spread over it
            Acc acc[NT][NB];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[t][j] = Acc{0, 0, 0, 0};
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                if (s + 1 < nch) fetch(it, QT ? ch + 1 : ch - 1, rt);
                else if (more) fetch(nx, QT ? 0 : nx.nch - 1, rt);
                T a[NT][4];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    constexpr int kPer = 16 / sizeof(T);
#pragma unroll
                    for (int h = 0; h < 4; h += kPer) {
                        typedef T Piece __attribute__((ext_vector_type(kPer)));
                        const Piece p = *reinterpret_cast<const Piece *>(
                            &Vw[16 * t + l16][row_place<T>(16 * rt + 4 * l4 + h, l16)]);
#pragma unroll
                        for (int i = 0; i < kPer; ++i) a[t][h + i] = p[i];
                    }
                }
                Acc part[NT][NB];
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int j = 0; j < NB; ++j) part[t][j] = kTileSums ? Acc{0, 0, 0, 0} : acc[t][j];
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        const T x = T(b[rt][j][r]);
#pragma unroll
                        for (int t = 0; t < NT; ++t) part[t][j] = Tile::mfma(a[t][r], x, part[t][j]);
                    }
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int j = 0; j < NB; ++j) acc[t][j] = kTileSums ? acc[t][j] + part[t][j] : part[t][j];
                __builtin_amdgcn_sched_barrier(0);
            }
            // the partials meet: W's rows 16 w .. on wave w
            Acc wv[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                __syncthreads();
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (t == w) wv[j] = acc[t][j];
                    else red[3 * t + (w < t ? w : w - 1)][lane] = acc[t][j];
                }
                __syncthreads();
                if (own) {
                    wv[j] = wv[j] + red[3 * w][lane] + red[3 * w + 1][lane] + red[3 * w + 2][lane];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (!first) wv[j][r] += T(y[j][r]);
                        wv[j][r] = 16 * w + Tile::drow(r, lane) < n ? wv[j][r] : T(0);
                    }
                }
            }
            __syncthreads();
            if (own) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) Wx[16 * w + Tile::drow(r, lane)][16 * j + l16] = wv[j][r];
            }
            __syncthreads();
            Acc z[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) z[j] = Acc{0, 0, 0, 0};
            if (own) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (QT ? t <= w : t >= w) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            bool ok;
                            t_at(t, u, ok);
                            const T a = ok ? T(tk[t][u]) : T(0);
#pragma unroll
                            for (int j = 0; j < NB; ++j)
                                z[j] = Tile::mfma(a, Wx[16 * t + 4 * u + l4][16 * j + l16], z[j]);
                        }
                    }
            }
            __syncthreads();
            if (own) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (!first) y[j][r] -= (double)z[j][r];
                        Wx[16 * w + Tile::drow(r, lane)][16 * j + l16] = -z[j][r];
                    }
            }
            __syncthreads();
            T zb[NT][4][NB];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int j = 0; j < NB; ++j) zb[t][u][j] = Wx[16 * t + 4 * u + l4][16 * j + l16];
            __syncthreads();
            asm volatile("" : "+v"(lane));
            l16 = lane & 15;
            l4 = lane >> 4;
            // B - V Z
            const int prow = tile_row_of<Tile>(l16);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                Acc c[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) c[j] = Acc{0, 0, 0, 0};
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int col = 16 * t + 4 * u + l4;
                        const T a = Vw[col][row_place<T>(16 * rt + prow, 4 * u + l4)];
#pragma unroll
                        for (int j = 0; j < NB; ++j) c[j] = Tile::mfma(a, zb[t][u][j], c[j]);
                    }
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        b[rt][j][r] += (double)c[j][r];
                        // now, not behind the next branch with every product kept for it
                        asm volatile("" : "+v"(b[rt][j][r]));
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (first && QT) {   // Yb starts as a first chunk's top rows
                if (w == 0) {
#pragma unroll
                    for (int rt = 0; rt < NT; ++rt)
#pragma unroll
                        for (int j = 0; j < NB; ++j)
#pragma unroll
                            for (int r = 0; r < 4; ++r) Yx[16 * rt + 4 * l4 + r][16 * j + l16] = b[rt][j][r];
                }
                __syncthreads();
                if (own) {
#pragma unroll
                    for (int j = 0; j < NB; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r) y[j][r] = Yx[16 * w + Tile::drow(r, lane)][16 * j + l16];
                }
                __syncthreads();
            }
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" : "+v"(lane));
            l16 = lane & 15;
            l4 = lane >> 4;
            const int lo = (first && QT && w == 0) ? n : 0;   // rows that became Yb
#pragma unroll
            for (int j = 0; j < NB; ++j) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int h = 0; h < 4; h += 2)
                        *reinterpret_cast<double2 *>(&Bw[l16][row_place<double>(16 * rt + 4 * l4 + h, l16)]) =
                            double2{b[rt][j][h], b[rt][j][h + 1]};
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int r = 64 * h + lane;
                    double o[16];
#pragma unroll
                    for (int c = 0; c < 16; ++c) o[c] = Bw[c][row_place<double>(r, c)];
                    if (16 * RT * w + r < valid && r >= lo) {
#pragma unroll
                        for (int c = 0; c < 16; ++c)
                            if (16 * j + c < kc) (B + off + (int64_t)(16 * j + c) * ldb)[16 * RT * w + r] = o[c];
                    }
                }
            }
        }
        if constexpr (QT) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * w + Tile::drow(r, lane), c = 16 * j + l16;
                    if (c < kc && row < n) B[row + (int64_t)c * ldb] = y[j][r];
                }
        }
        if (!more) return;
        it = nx;
    }
}

template <typename Tile, int NT, int NB, bool LOW, bool QT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_leaf_apply_m(const typename Tile::T *__restrict__ V, int64_t ldv, const double *__restrict__ Tc,
                    PanelArgs pa, const double *Bsrc, int64_t ldbs, double *B, int64_t ldb, int64_t k, int ncb) {
    extern __shared__ __attribute__((aligned(64))) unsigned char smem_bytes[];
    auto &sm = *reinterpret_cast<LeafApplySmem<Tile, NT, NB, LOW> *>(smem_bytes);
    leaf_apply_chains<Tile, NT, NB, LOW, QT>(sm, V, ldv, Tc, pa, Bsrc, ldbs, B, ldb, k, ncb);
}

// As many workgroups as the compute units hold (by LDS).
template <typename Tile, int NT, int NB, bool LOW, bool QT>
static hipError_t launch_apply_m(const typename Tile::T *V, int64_t ldv, const double *Tc, const PanelArgs &pa,
                                 const double *Bsrc, int64_t ldbs, double *B, int64_t ldb, int64_t k,
                                 const char *tag, hipStream_t st) {
    const size_t sh = sizeof(LeafApplySmem<Tile, NT, NB, LOW>);
    const auto kern = k_leaf_apply_m<Tile, NT, NB, LOW, QT>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    const int ncb = (int)((k + 16 * NB - 1) / (16 * NB));
    const int64_t items = (pa.P + 7) / 8 * 8 * ncb, cap = kComputeUnits * (int64_t)(160 * 1024 / sh);
    ProfScope ps(tag, st);
    hipLaunchKernelGGL(kern, dim3((unsigned)(items < cap ? items : cap)), dim3(256), sh, st, V, ldv, Tc, pa, Bsrc,
                       ldbs, B, ldb, k, ncb);
    return hipGetLastError();
}

// 32 columns per workgroup read V half as often and share each of its LDS
// reads between two tiles, but only where that still gives every compute
// unit a workgroup: a chunk then takes 30 thousand cycles against 2 x 21.
template <typename Tile>
static hipError_t launch_apply_m(const typename Tile::T *V, int64_t ldv, const double *Tc, const PanelArgs &pa,
                                 const double *Bsrc, int64_t ldbs, double *B, int64_t ldb, int64_t k, int trans,
                                 const char *tag, hipStream_t st) {
    if (k <= 0) return hipSuccess;
    const bool wide = k > 16 && pa.P * ((k + 31) / 32) >= kComputeUnits;
    // Low domains have their own form for FP32 reflectors, where it keeps bits
    // (error of Q Q^T B, 200,001 rows in domains of 64: 40 columns 7.9e-4 -> 6.0e-4,
    // 16 columns 4.9e-4 -> 3.1e-4, at 3 % of the time), and up to 16 columns, whose
    // chunks are 512 rows: half of the registers and LDS (100,003 x 8 in domains of 8
    // rows, 17 columns 0.93 -> 0.71 ms).  Wider FP64 ones would spill (64 columns
    // in domains of 64 rows, 17 columns of B: 0.49 -> 0.92 ms).
    const bool low = !pa.wtab && !pa.extra && 2 * pa.mb <= pa.chunk && 2 * dom_rows(pa, pa.P - 1) <= pa.chunk;
    auto go = [&](auto nt, auto nb, auto qt) {
        constexpr int NT = decltype(nt)::value, NB = decltype(nb)::value;
        constexpr bool QT = decltype(qt)::value;
        if constexpr (NT == 1 || sizeof(typename Tile::T) == 4) {
            if (low) return launch_apply_m<Tile, NT, NB, true, QT>(V, ldv, Tc, pa, Bsrc, ldbs, B, ldb, k, tag, st);
        }
        return launch_apply_m<Tile, NT, NB, false, QT>(V, ldv, Tc, pa, Bsrc, ldbs, B, ldb, k, tag, st);
    };
    auto with_nt = [&](auto nb, auto qt) {
        switch ((pa.n + 15) >> 4) {
            case 1: return go(std::integral_constant<int, 1>{}, nb, qt);
            case 2: return go(std::integral_constant<int, 2>{}, nb, qt);
            case 3: return go(std::integral_constant<int, 3>{}, nb, qt);
            default: return go(std::integral_constant<int, 4>{}, nb, qt);
        }
    };
    auto with_nb = [&](auto qt) {
        return wide ? with_nt(std::integral_constant<int, 2>{}, qt) : with_nt(std::integral_constant<int, 1>{}, qt);
    };
    return trans ? with_nb(std::true_type{}) : with_nb(std::false_type{});
}

hipError_t launch_leaf_apply_m(const double *V, int64_t ldv, const double *Tc, const PanelArgs &pa,
                               const double *Bsrc, int64_t ldbs, double *B, int64_t ldb, int64_t k,
                               int trans, hipStream_t st) {
    return launch_apply_m<TileF64>(V, ldv, Tc, pa, Bsrc, ldbs, B, ldb, k, trans,
                                   trans ? "leaf_apply_qt" : "leaf_apply_q", st);
}

hipError_t launch_leaf_apply_m32(const float *V, int64_t ldv, const double *Tc, const PanelArgs &pa,
                                 const double *Bsrc, int64_t ldbs, double *B, int64_t ldb, int64_t k,
                                 int trans, hipStream_t st) {
    return launch_apply_m<TileF32>(V, ldv, Tc, pa, Bsrc, ldbs, B, ldb, k, trans,
                                   trans ? "leaf_apply_qt_f32" : "leaf_apply_q_f32", st);
}

// ---------------------------------------------------------------------------
// Three-pass leaf apply for few columns (k <= 16).  The chunk chain of a
// domain couples chunks only through the n x k running top rows Y, so
//   pass 1 (every chunk at once):  P_c = V_c^T B_c            (a first chunk
//                                  from row n on: its top rows are Y)
//   pass 2 (one workgroup/domain): the chain on n x k blocks,
//          Q^T: W_0 = V_0top^T Y + P_0, Z_0 = T_0^T W_0, Y <- Y - V_0top Z_0,
//               then W_c = Y + P_c, Z_c = T_c^T W_c, Y <- Y - Z_c (c = 1..),
//          Q:   chunks last to first with T_c, chunk 0 last, top rows
//               written as Y - V_0top Z_0;
//   pass 3 (every chunk at once):  B_c <- B_c - V_c Z_c   (rows below the
//                                  top rows of a first chunk).
// V is streamed twice across the whole device instead of once chunk after
// chunk; the chain touches only T and n x k blocks.  P_c and Z_c are n x k
// column-major blocks, one per chunk.

// Rows [rlo, valid) of chunk c: W(n x kc) = V_c^T B_c, one partial per wave
// in sm.Wp (tile precision); the caller adds the four in wave order.
template <typename Tile>
struct VtbSmem {
    using T = typename Tile::T;
    // per-wave partials of V^T B, entry (wave w, row m, column j < kc) at
    // (64 w + m) kc + j: a launch sizes the LDS by its own kc (vtb_lds_bytes)
    T Wp[4 * 64 * KBM];
};
template <typename Tile>
constexpr size_t vtb_lds_bytes(int64_t kc) {
    return (size_t)4 * 64 * (size_t)kc * sizeof(typename Tile::T);
}

// Four consecutive rows of a column, at any alignment of the element's.
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void load_rows4(const double *__restrict__ p, double (&v)[4]) {
    const d2u a = *reinterpret_cast<const d2u *>(p), b = *reinterpret_cast<const d2u *>(p + 2);
    v[0] = a.x;
    v[1] = a.y;
    v[2] = b.x;
    v[3] = b.y;
}
__device__ __forceinline__ void load_rows4(const float *__restrict__ p, float (&v)[4]) {
    const f4u a = *reinterpret_cast<const f4u *>(p);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = a[q];
}

// n <= 16 NT.  A lane reads 4 consecutive rows of its column (16 rows x 16
// columns per load); MFMA q takes row 4 l4 + q of the block as its k = l4
// element.  Two blocks' loads go out together, with no condition on them:
// columns past the last repeat it (their products are dropped), and so do
// rows, against zeros of B.  What bounds it: reading V.  With loads that needed
// 16-byte column starts (element loads elsewhere) and a condition each, odd
// heights ran at a quarter of the rate: 32 mixed matrices of 1,000 to 200,000
// rows 350 -> 150 us, 1,048,576 x 64 FP32 66 -> 60 us.
template <typename Tile, int NT>
__device__ __forceinline__ void chunk_vtb(VtbSmem<Tile> &sm, const typename Tile::T *__restrict__ Vc,
                                          int64_t ldv, const double *__restrict__ Bc, int64_t ldb,
                                          int rlo, int valid, int n, int kc) {
    using T = typename Tile::T;
    using Acc = typename Tile::Acc;
    const int lane = threadIdx.x & 63, w = wave_index<4>(), l16 = lane & 15, l4 = lane >> 4;
    Acc acc[NT];
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) acc[mt] = Acc{0, 0, 0, 0};
    const int span = valid - rlo, per = ((span + 15) / 16 + 3) / 4 * 16;
    const int lo = rlo + w * per, hi = (lo + per < valid) ? lo + per : valid;
    const double *bp = Bc + (int64_t)(l16 < kc ? l16 : kc - 1) * ldb;
    const T *vp[NT];
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) vp[mt] = Vc + (int64_t)(16 * mt + l16 < n ? 16 * mt + l16 : n - 1) * ldv;
    int r16 = lo;
#pragma unroll 1
    for (; r16 + 32 <= hi; r16 += 32) {
        double b[2][4];
        T a[2][NT][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int rb = r16 + 16 * u + 4 * l4;
            load_rows4(bp + rb, b[u]);
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) load_rows4(vp[mt] + rb, a[u][mt]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int mt = 0; mt < NT; ++mt) acc[mt] = Tile::mfma(a[u][mt][q], T(b[u][q]), acc[mt]);
    }
#pragma unroll 1
    for (; r16 < hi; r16 += 16) {
        double b[4];
        T a[NT][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = r16 + 4 * l4 + q, rc = r < hi ? r : hi - 1;
            b[q] = bp[rc];
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) a[mt][q] = vp[mt][rc];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const T x = r16 + 4 * l4 + q < hi ? T(b[q]) : T(0);
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) acc[mt] = Tile::mfma(a[mt][q], x, acc[mt]);
        }
    }
    if (l16 < kc) {
#pragma unroll
        for (int mt = 0; mt < NT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) sm.Wp[(64 * w + 16 * mt + Tile::drow(r, lane)) * kc + l16] = acc[mt][r];
    }
    __syncthreads();
}

template <typename Tile>
__device__ __forceinline__ void apply_p1_body(const typename Tile::T *__restrict__ V, int64_t ldv,
                                              const PanelArgs &pa, const double *__restrict__ B, int64_t ldb,
                                              int64_t k, double *__restrict__ Pc, int64_t dom, int64_t ch) {
    extern __shared__ double smem_raw[];
    VtbSmem<Tile> &sm = *reinterpret_cast<VtbSmem<Tile> *>(smem_raw);
    const int n = pa.n;
    const int64_t row0 = dom_row0(pa, dom);
    const int64_t nrows = dom_rows(pa, dom);
    const int64_t nch = (nrows + pa.chunk - 1) / pa.chunk;
    if (ch >= nch) return;
    const int kc = (int)k;
    const int64_t r0 = row0 + ch * pa.chunk;
    const int valid = (int)((nrows - ch * pa.chunk < pa.chunk) ? nrows - ch * pa.chunk : pa.chunk);
    auto vtb = [&](auto nt) {
        chunk_vtb<Tile, decltype(nt)::value>(sm, V + r0, ldv, B + r0, ldb, ch == 0 ? n : 0, valid, n, kc);
    };
    switch ((n + 15) >> 4) {
        case 1: vtb(std::integral_constant<int, 1>{}); break;
        case 2: vtb(std::integral_constant<int, 2>{}); break;
        case 3: vtb(std::integral_constant<int, 3>{}); break;
        default: vtb(std::integral_constant<int, 4>{});
    }
    // P_c = the four waves' partials added in wave order
    using T = typename Tile::T;
    double *P = Pc + (dom_chunk0(pa, dom) + ch) * (int64_t)n * k;
    const int ws = 64 * kc;
    for (int e = threadIdx.x; e < n * kc; e += 256) {
        const int m = e % n, j = e / n, o = m * kc + j;
        const T sum = ((sm.Wp[o] + sm.Wp[ws + o]) + sm.Wp[2 * ws + o]) + sm.Wp[3 * ws + o];
        P[e] = (double)sum;
    }
}

template <typename Tile>
__global__ __launch_bounds__(256) void k_apply_p1(const typename Tile::T *__restrict__ V, int64_t ldv,
                                                  PanelArgs pa, const double *__restrict__ B, int64_t ldb,
                                                  int64_t k, double *__restrict__ Pc) {
    apply_p1_body<Tile>(V, ldv, pa, B, ldb, k, Pc, blockIdx.y, blockIdx.x);
}

template <int NT>
struct ChainSmem {
    double W[2][16 * NT][KBM];
    double Z[16 * NT][KBM];
};

// Pass 2 for one domain (FP64), n <= 16 NT: wave w owns rows 16 w .. 16 w + 15
// of Y (in registers for the whole chain), W and Z; T's operand and P_c come
// from memory a chunk ahead, W crosses the waves through LDS (two buffers:
// one barrier a chunk).  What bounds it: the chain -- per chunk 16 dependent
// matrix-core tiles of 64 cycles and the barrier -- and reading T.  Measured at 16 chunks of 64
// columns: 81 -> 45 us, against dot products of up to 64 terms per thread.
template <bool QT, int NT>
__device__ __forceinline__ void apply_p2_chain(ChainSmem<NT> &sm, const double *__restrict__ V64,
                                               const float *__restrict__ V32, int64_t ldv,
                                               const double *__restrict__ Tc, const PanelArgs &pa,
                                               double *__restrict__ B, int64_t ldb, int64_t k,
                                               const double *__restrict__ Pc, double *__restrict__ Zc, int64_t dom) {
    const int n = pa.n, kc = (int)k;
    const int w = wave_index<4>(), lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
    const int64_t nn = (int64_t)n * n, row0 = dom_row0(pa, dom), nrows = dom_rows(pa, dom);
    const int64_t nch = (nrows + pa.chunk - 1) / pa.chunk;
    const double *T0 = Tc + dom_chunk0(pa, dom) * nn;
    const double *P0 = Pc + dom_chunk0(pa, dom) * (int64_t)n * k;
    double *Z0 = Zc + dom_chunk0(pa, dom) * (int64_t)n * k;
    const bool own = w < NT, colok = l16 < kc;
    const int col = colok ? l16 : 0;
    auto row_of = [&](int r) { return 16 * w + 4 * r + l4; };
    // op(T)'s entry kb of this lane: (4 kb + l4, 16 w + l16) or, for Q, its transpose's place
    auto t_at = [&](int kb, bool &ok) {
        const int i = 16 * w + l16, q = 4 * kb + l4, r = QT ? q : i, c = QT ? i : q;
        ok = r <= c && c < n;
        return ok ? r + c * n : 0;
    };
    // V_0top's entry (r, c), unit lower triangular
    auto v0 = [&](int r, int c) {
        const bool ok = c < r && r < n;
        const int64_t at = row0 + (ok ? r + (int64_t)c * ldv : 0);
        const double v = V32 ? (double)V32[at] : V64[at];
        return r == c ? 1.0 : (ok ? v : 0.0);
    };
    // T's operand and P_c of the next chunk
    double tn[4 * NT];
    d4 pn;
    auto fetch = [&](int64_t ch) {
#pragma unroll
        for (int kb = 0; kb < 4 * NT; ++kb) {
            bool ok;
            tn[kb] = T0[ch * nn + t_at(kb, ok)];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            pn[r] = P0[ch * (int64_t)n * k + (row_of(r) < n ? row_of(r) : 0) + (int64_t)col * n];
    };
    auto chunk_of_step = [&](int64_t s) {   // past the chain: its last chunk again (not used)
        s = s < nch ? s : nch - 1;
        return QT ? s : nch - 1 - s;
    };
    fetch(chunk_of_step(0));
    d4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double v = B[row0 + (row_of(r) < n ? row_of(r) : 0) + (int64_t)col * ldb];
        y[r] = (colok && row_of(r) < n) ? v : 0.0;
    }
    // step s: `add` to P_c gives W, then Z = op(T) W
    auto zed = [&](int64_t s, const d4 &add) {
        const int64_t ch = chunk_of_step(s);
        double(*W)[KBM] = sm.W[s & 1];
        double t[4 * NT];
#pragma unroll
        for (int kb = 0; kb < 4 * NT; ++kb) {
            bool ok;
            t_at(kb, ok);
            t[kb] = ok ? tn[kb] : 0.0;
        }
        if (own) {
#pragma unroll
            for (int r = 0; r < 4; ++r) W[row_of(r)][l16] = row_of(r) < n ? (colok ? pn[r] : 0.0) + add[r] : 0.0;
        }
        fetch(chunk_of_step(s + 1));
        __syncthreads();
        d4 z = d4_zero();
        if (own) {
#pragma unroll
            for (int kb = 0; kb < 4 * NT; ++kb) z = mfma_f64(t[kb], W[4 * kb + l4][l16], z);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (colok && row_of(r) < n) Z0[ch * (int64_t)n * k + row_of(r) + (int64_t)col * n] = z[r];
        }
        return z;
    };
    // the first chunk: W = V_0top^T Y + P, Y <- Y - V_0top Z
    auto first = [&](int64_t s) {
        d4 acc = d4_zero();
        if (own) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sm.Z[row_of(r)][l16] = y[r];
        }
        __syncthreads();
        if (own) {
            double a[4 * NT];
#pragma unroll
            for (int kb = 0; kb < 4 * NT; ++kb) a[kb] = v0(4 * kb + l4, 16 * w + l16);
#pragma unroll
            for (int kb = 0; kb < 4 * NT; ++kb) acc = mfma_f64(a[kb], sm.Z[4 * kb + l4][l16], acc);
        }
        const d4 z = zed(s, acc);
        if (own) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sm.Z[row_of(r)][l16] = z[r];
        }
        __syncthreads();
        if (own) {
            double a[4 * NT];
#pragma unroll
            for (int kb = 0; kb < 4 * NT; ++kb) a[kb] = v0(16 * w + l16, 4 * kb + l4);
            acc = d4_zero();
#pragma unroll
            for (int kb = 0; kb < 4 * NT; ++kb) acc = mfma_f64(a[kb], sm.Z[4 * kb + l4][l16], acc);
            y -= acc;
        }
    };
    if constexpr (QT) first(0);
#pragma unroll 1
    for (int64_t s = QT ? 1 : 0; s < (QT ? nch : nch - 1); ++s) y -= zed(s, y);
    if constexpr (!QT) first(nch - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (colok && row_of(r) < n) B[row0 + row_of(r) + (int64_t)col * ldb] = y[r];
}

template <bool QT>
__device__ __forceinline__ void apply_p2_body(const double *__restrict__ V64, const float *__restrict__ V32,
                                              int64_t ldv, const double *__restrict__ Tc, const PanelArgs &pa,
                                              double *__restrict__ B, int64_t ldb, int64_t k,
                                              const double *__restrict__ Pc, double *__restrict__ Zc, int64_t dom) {
    __shared__ ChainSmem<4> sm;
    auto run = [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        apply_p2_chain<QT, NT>(reinterpret_cast<ChainSmem<NT> &>(sm), V64, V32, ldv, Tc, pa, B, ldb, k, Pc, Zc, dom);
    };
    switch ((pa.n + 15) >> 4) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        default: run(std::integral_constant<int, 4>{});
    }
}

template <bool QT>
__global__ __launch_bounds__(256) void k_apply_p2(const double *__restrict__ V64, const float *__restrict__ V32,
                                                  int64_t ldv, const double *__restrict__ Tc, PanelArgs pa,
                                                  double *__restrict__ B, int64_t ldb, int64_t k,
                                                  const double *__restrict__ Pc, double *__restrict__ Zc) {
    apply_p2_body<QT>(V64, V32, ldv, Tc, pa, B, ldb, k, Pc, Zc, blockIdx.x);
}

// Pass 3: B_c <- B_c - V_c Z_c over the chunk's rows (a first chunk from
// row n on), transposed: a product tile's columns are 16 rows of B.  A lane
// reads two consecutive rows of V (32 rows x 4 columns per load), one for each
// of two tiles; the Z operand stays in registers, so the kernel needs no LDS
// and many workgroups share a CU.  The loads are unconditional: columns past
// the last repeat it and meet zeros of Z, a pair of rows past the end moves
// back to the last two.  What bounds it: reading V.  Against one row a lane and
// a condition on each load: 32 mixed matrices of 1,000 to 200,000 rows 235 ->
// 155 us, 1,048,576 x 64 FP64 134 -> 120 us.
template <typename T>
struct RowPair;
template <>
struct RowPair<double> { using V = d2u; };
template <>
struct RowPair<float> { using V = f2u; };

template <typename Tile, int NT>
__device__ __forceinline__ void chunk_minus_vz(const typename Tile::T *__restrict__ Vc, int64_t ldv,
                                               double *__restrict__ Bc, int64_t ldb, const double *__restrict__ Z,
                                               int64_t r0, int lo, int valid, int n, int kc) {
    using T = typename Tile::T;
    using Acc = typename Tile::Acc;
    using Pair = typename RowPair<T>::V;
    const int lane = threadIdx.x & 63, w = wave_index<4>(), l16 = lane & 15, l4 = lane >> 4;
    // A[i][q] = Z^T[col i][reflector q] for q = 4 kb + l4
    T za[4 * NT];
#pragma unroll
    for (int kb = 0; kb < 4 * NT; ++kb) {
        const int q = 4 * kb + l4;
        const bool ok = q < n && l16 < kc;
        const double z = Z[ok ? q + l16 * n : 0];
        za[kb] = ok ? T(z) : T(0);
    }
#pragma unroll 1
    for (int t0 = 32 * w; t0 < valid; t0 += 128) {
        const int R = t0 + 2 * l16;
        int Rc = R < valid - 2 ? R : valid - 2;
        if (r0 == 0 && Rc < 0) Rc = 0;   // one row in all: the pair's second is not used
        const T *vp = Vc + Rc;
        Pair v[4 * NT];
#pragma unroll
        for (int kb = 0; kb < 4 * NT; ++kb)
            v[kb] = *reinterpret_cast<const Pair *>(vp + (int64_t)(4 * kb + l4 < n ? 4 * kb + l4 : n - 1) * ldv);
        Acc acc[2] = {Acc{0, 0, 0, 0}, Acc{0, 0, 0, 0}};
        if (Rc != R) {   // a moved pair's second row is row R, where there is one
#pragma unroll
            for (int kb = 0; kb < 4 * NT; ++kb) v[kb].x = v[kb].y;
        }
#pragma unroll
        for (int kb = 0; kb < 4 * NT; ++kb) {
            acc[0] = Tile::mfma(za[kb], v[kb].x, acc[0]);
            acc[1] = Tile::mfma(za[kb], v[kb].y, acc[1]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int col = Tile::drow(r, lane);
            if (col < kc) {
                double *p = Bc + R + (int64_t)col * ldb;
                if (R >= lo && R < valid) p[0] -= (double)acc[0][r];
                if (R + 1 >= lo && R + 1 < valid) p[1] -= (double)acc[1][r];
            }
        }
    }
}

template <typename Tile>
__device__ __forceinline__ void apply_p3_body(const typename Tile::T *__restrict__ V, int64_t ldv,
                                              const PanelArgs &pa, double *__restrict__ B, int64_t ldb, int64_t k,
                                              const double *__restrict__ Zc, int64_t dom, int64_t ch) {
    const int n = pa.n, kc = (int)k;
    const int64_t row0 = dom_row0(pa, dom);
    const int64_t nrows = dom_rows(pa, dom);
    const int64_t nch = (nrows + pa.chunk - 1) / pa.chunk;
    if (ch >= nch) return;
    const int64_t r0 = row0 + ch * pa.chunk;
    const int valid = (int)((nrows - ch * pa.chunk < pa.chunk) ? nrows - ch * pa.chunk : pa.chunk);
    const double *Z = Zc + (dom_chunk0(pa, dom) + ch) * (int64_t)n * k;
    auto run = [&](auto nt) {
        chunk_minus_vz<Tile, decltype(nt)::value>(V + r0, ldv, B + r0, ldb, Z, r0, ch == 0 ? n : 0, valid, n, kc);
    };
    switch ((n + 15) >> 4) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        default: run(std::integral_constant<int, 4>{});
    }
}

template <typename Tile>
__global__ __launch_bounds__(256) void k_apply_p3(const typename Tile::T *__restrict__ V, int64_t ldv,
                                                  PanelArgs pa, double *__restrict__ B, int64_t ldb, int64_t k,
                                                  const double *__restrict__ Zc) {
    apply_p3_body<Tile>(V, ldv, pa, B, ldb, k, Zc, blockIdx.y, blockIdx.x);
}

// ---- batched forms on each listed matrix's vector F (k = 1); grid.x walks
// the matrix's chunks (pass 1, 3) or domains (pass 2); sweep > 0 skips
// converged matrices.
__device__ __forceinline__ bool chunk_of(const BMat &M, int64_t g, int64_t &dom, int64_t &ch) {
    if (g >= M.tchunks) return false;
    dom_of_chunk(M.pa, g, dom, ch);
    return true;
}

// MIXED: only mixed matrices are listed (every refinement sweep's list): the
// FP64 form's registers would halve the waves in flight.
template <bool MIXED>
__global__ __launch_bounds__(256) void k_apply_p1_b(const BMat *__restrict__ mats, const int *__restrict__ list,
                                                    int sweep) {
    const BMat &M = mats[list[blockIdx.y]];
    int64_t dom, ch;
    if (!chunk_of(M, blockIdx.x, dom, ch)) return;
    if (sweep > 0 && M.status[1]) return;
    if (MIXED || M.prec) apply_p1_body<TileF32>(M.V32, M.pa.m, M.pa, M.F, M.pa.m, 1, M.Pc, dom, ch);
    else apply_p1_body<TileF64>(M.V, M.pa.m, M.pa, M.F, M.pa.m, 1, M.Pc, dom, ch);
}

template <bool QT>
__global__ __launch_bounds__(256) void k_apply_p2_b(const BMat *__restrict__ mats, const int *__restrict__ list,
                                                    int sweep) {
    const BMat &M = mats[list[blockIdx.y]];
    if ((int64_t)blockIdx.x >= M.pa.P) return;
    if (sweep > 0 && M.status[1]) return;
    apply_p2_body<QT>(M.V, M.V32, M.pa.m, M.Tc, M.pa, M.F, M.pa.m, 1, M.Pc, M.Zc, blockIdx.x);
}

template <bool MIXED>
__global__ __launch_bounds__(256) void k_apply_p3_b(const BMat *__restrict__ mats, const int *__restrict__ list,
                                                    int sweep) {
    const BMat &M = mats[list[blockIdx.y]];
    int64_t dom, ch;
    if (!chunk_of(M, blockIdx.x, dom, ch)) return;
    if (sweep > 0 && M.status[1]) return;
    if (MIXED || M.prec) apply_p3_body<TileF32>(M.V32, M.pa.m, M.pa, M.F, M.pa.m, 1, M.Zc, dom, ch);
    else apply_p3_body<TileF64>(M.V, M.pa.m, M.pa, M.F, M.pa.m, 1, M.Zc, dom, ch);
}

hipError_t launch_apply3_b(const BMat *mats, const int *list, int cnt, int64_t max_chunks, int64_t max_p,
                           int trans, int sweep, hipStream_t st) {
    if (cnt <= 0 || max_chunks <= 0) return hipSuccess;
    const size_t sh = vtb_lds_bytes<TileF64>(1);   // k = 1
    const auto p1 = sweep > 0 ? k_apply_p1_b<true> : k_apply_p1_b<false>;
    const auto p3 = sweep > 0 ? k_apply_p3_b<true> : k_apply_p3_b<false>;
    hipError_t e = hipFuncSetAttribute((const void *)p1, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    {
        ProfScope ps(trans ? "batch_apply3_p1_qt" : "batch_apply3_p1_q", st);
        hipLaunchKernelGGL(p1, dim3((unsigned)max_chunks, (unsigned)cnt), dim3(256), sh, st, mats, list, sweep);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    {
        ProfScope ps(trans ? "batch_apply3_p2_qt" : "batch_apply3_p2_q", st);
        const auto kern = trans ? k_apply_p2_b<true> : k_apply_p2_b<false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)max_p, (unsigned)cnt), dim3(256), 0, st, mats, list, sweep);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    ProfScope ps(trans ? "batch_apply3_p3_qt" : "batch_apply3_p3_q", st);
    hipLaunchKernelGGL(p3, dim3((unsigned)max_chunks, (unsigned)cnt), dim3(256), 0, st, mats, list, sweep);
    return hipGetLastError();
}

template <typename Tile>
static hipError_t launch_apply3(const typename Tile::T *V, const double *V64, const float *V32, int64_t ldv,
                                const double *Tc, const PanelArgs &pa, double *B, int64_t ldb, int64_t k,
                                int trans, double *Pc, double *Zc, hipStream_t st) {
    if (k <= 0) return hipSuccess;
    const size_t sh = vtb_lds_bytes<Tile>(k);
    hipError_t e = hipFuncSetAttribute((const void *)k_apply_p1<Tile>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    if (e != hipSuccess) return e;
    const dim3 chunks((unsigned)max_domain_chunks(pa), (unsigned)pa.P);
    {
        ProfScope ps(trans ? "apply3_p1_qt" : "apply3_p1_q", st);
        hipLaunchKernelGGL(k_apply_p1<Tile>, chunks, dim3(256), sh, st, V, ldv, pa, B, ldb, k, Pc);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    {
        ProfScope ps(trans ? "apply3_p2_qt" : "apply3_p2_q", st);
        const auto kern = trans ? k_apply_p2<true> : k_apply_p2<false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)pa.P), dim3(256), 0, st, V64, V32, ldv, Tc, pa, B, ldb, k, Pc, Zc);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    ProfScope ps(trans ? "apply3_p3_qt" : "apply3_p3_q", st);
    hipLaunchKernelGGL(k_apply_p3<Tile>, chunks, dim3(256), 0, st, V, ldv, pa, B, ldb, k, Zc);
    return hipGetLastError();
}

hipError_t launch_leaf_apply3(const double *V, int64_t ldv, const double *Tc, const PanelArgs &pa, double *B,
                              int64_t ldb, int64_t k, int trans, double *Pc, double *Zc, hipStream_t st) {
    return launch_apply3<TileF64>(V, V, nullptr, ldv, Tc, pa, B, ldb, k, trans, Pc, Zc, st);
}

hipError_t launch_leaf_apply3_32(const float *V, int64_t ldv, const double *Tc, const PanelArgs &pa,
                                 double *B, int64_t ldb, int64_t k, int trans, double *Pc, double *Zc,
                                 hipStream_t st) {
    return launch_apply3<TileF32>(V, nullptr, V, ldv, Tc, pa, B, ldb, k, trans, Pc, Zc, st);
}

}  // namespace tsqr
