// Factorization level step with one workgroup per node for block sizes
// n <= 64, every block in registers as 16 x 16 tiles (NTL of them a side, as many
// as n needs: every tile row holds rows of the block).
//
// Per node i of level l (stride s, h = s/2; Algorithm 4, hybrid left/right-
// looking, deterministic ownership):
//   1  S_i     -= T'^T T'     T'  = T_{i+h}    (deferred from level l-1)
//      S_{i+s} -= T''^T T''   T'' = T_{i+3h}
//   2  L_ii = chol(S_i);  R_i = C_{i+s,i} L_ii^{-T},  T_i = L_ii^{-1} C_{i,i-s}
//   3  S_{i+s} -= R_i R_i^T,  fill -R_i T_i.
//
// Step 2 is one tall panel factorization: the rows of C_{i+s,i} and of
// C_{i,i-s}^T are rows below S_i, so R_i and T_i^T come out of the same
// 4-column steps as L_ii (panel_step).  Wavefront w of NTL = NP/16 carries
// tile-row w of R_i, tile-column w of T_i and tile-row w of L_ii; each repeats
// the steps of the diagonal tile, so that none waits on another inside a
// panel.
//
// Nothing is laid out anew between the steps.  A tile in four registers,
// register v of lane l holding element (l % 16, 4v + l / 16) of the tile, is
//   the A operand of v_mfma_*_16x16x4 for the four k chunks (X of X Y),
//   the B operand for its transpose (Y = X^T), and
//   the FP64 accumulator of its transpose,
// so S_i, the couplings, R_i and T_i^T are updated, solved and multiplied in that
// one form; LDS passes tiles between wavefronts and turns those whose rows lie
// across the lanes (C_{i+s,i}, R_i, L_ii), so that loads and stores cover four
// rows of 16 elements instead of sixteen rows of 4.
//
// What bounds it: large launches the memory (level 0 of N = 65 536, n = 32,
// FP64: 462 us for 72 KiB a node, 5.1 TB/s), small ones a node's own latency,
// of which the chains of 4-column steps are about a third, issuing the loads
// (all of them before the first use; from n = 33 on except T'') a fifth, the
// products the rest.  Measured against the kernels it replaces (blocks in LDS,
// the couplings' solves after the Cholesky factorization), one node of an
// inner level: n = 16 FP64 10.1 -> 7.1 us, n = 32 19.5 -> 11.9 (mixed, tile-
// parallel there: 16.4 -> 11.2), n = 8 (vector ALUs) 7.9 -> 6.7; at n = 33..64
// the tile-parallel step takes as long per node in FP64 (24.5 / 25.5 at n =
// 64) and longer in mixed precision (24.7 / 22.4), and is slower on wide levels
// (2048 nodes of n = 64: 157 / 139).  n = 33..48 has a kernel of three tile rows
// (N = 32 768, n = 48: 1 778 us with four, 1 594 with three; mixed 1 460, 1 318;
// an inner level 21.2 and 18.6).
//
// MODE 0: FP64.  MODE 1 (mixed precision): S_j, the Cholesky factorization and
// the triangular solves in FP64; L_ii, R_i, T_i and the fill rounded to FP32;
// Schur and fill products of the rounded blocks in FP32 (accumulated in FP32,
// subtracted in FP64).  MODE 2: as 1, the products with operands rounded to
// BF16 (nearest even).  What FP32 loses is won back by FP64 refinement.
#pragma once

#include <type_traits>

#include "btc_device.h"
#include "btc_kernels.h"
#include "btc_tiles.h"

namespace btc {
namespace node {

using namespace tiles;

// Tile products acc += (NEG ? -1 : 1) * A B over one 16-wide k tile: factor
// blocks of type F, accumulator of type Acc whose register v holds row
// row(v, lane / 16).
template <int MODE>
struct Prod {
    using F = float;
    using Acc = f4;
    __device__ static int row(int v, int q) { return 4 * q + v; }
    template <bool NEG>
    __device__ __forceinline__ static void tile(Acc& acc, const F (&a)[4], const F (&b)[4]) {
        if constexpr (MODE == 2) {
            typedef short s4 __attribute__((ext_vector_type(4)));
            typedef __bf16 h4 __attribute__((ext_vector_type(4)));
            h4 x, y;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                x[v] = (__bf16)(NEG ? -a[v] : a[v]);
                y[v] = (__bf16)b[v];
            }
            // k order 4 (lane / 16) + v instead of 4v + lane / 16, in both
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4, x), __builtin_bit_cast(s4, y), acc,
                                                            0, 0, 0);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(NEG ? -a[v] : a[v], b[v], acc, 0, 0, 0);
        }
    }
};
template <>
struct Prod<0> {
    using F = double;
    using Acc = d4;
    __device__ static int row(int v, int q) { return 4 * v + q; }
    template <bool NEG>
    __device__ __forceinline__ static void tile(Acc& acc, const F (&a)[4], const F (&b)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(NEG ? -a[v] : a[v], b[v], acc, 0, 0, 0);
    }
};

// X -= A B^T of FP64 tiles in the register form above (X as the accumulator
// of its transpose).
__device__ __forceinline__ void sub_abt(d4& x, const d4& a, const d4& b) {
#pragma unroll
    for (int v = 0; v < 4; ++v) x = __builtin_amdgcn_mfma_f64_16x16x4f64(-b[v], a[v], x, 0, 0, 0);
}

// A tile image in LDS: element (row, column) at 16 column + (row ^ column), so
// that both the register form (16 rows of 4 columns) and its transpose are
// read and written without bank conflicts.
constexpr int kImg = kT * kT;
__device__ __forceinline__ int img_pos(int row, int col) { return kT * col + (row ^ col); }

// Wavefronts per SIMD the register budget is set for: two workgroups of three
// or four wavefronts share a compute unit, four of two, twelve of one.
constexpr int node_waves(int ntl) { return ntl == 1 ? 3 : 2; }

template <int NTL, int MODE>
__global__ __launch_bounds__(NTL * kWave, node_waves(NTL)) void k_factor_node(Launch<FactorDesc> L) {
    using PR = Prod<MODE>;
    using F = typename PR::F;
    using Acc = typename PR::Acc;
    static_assert(NTL >= 1 && NTL <= 4, "tile rows");
    // tile pairs {w, (w + d) % NTL} of wavefront w cover the lower triangle
    constexpr int D = NTL / 2 + 1;
    constexpr int TB = NTL == 1 ? 2 : 3;  // tiles of a panel besides the diagonal one
    constexpr int kTri = NTL * (NTL + 1) / 2;
    // Three tile rows: the row of L_ii that a wavefront carries stays in LDS, in
    // S_i's images (four tile rows in FP64 have no room for those beside R_i's
    // and T_i's)
    constexpr bool kRowLds = NTL == 3;
    // LDS: images of R_i and T_i; from NTL = 3 on those of T' and T'' share
    // R_i's place, at NTL = 4 those of S_i start in T_i's, barriers between
    constexpr int kR = NTL == 1 ? 0 : NTL * NTL * kImg * (int)sizeof(F);
    constexpr int kS = kTri * kImg * 8;
    constexpr int kOverlay = kR + (NTL == 4 ? (kR > kS ? kR : kS) : kR + kS);
    constexpr int kL = NTL == 4 ? (NTL - 1 + NTL - 2 + 2) * kImg * 8 : 0;
    constexpr int kStage = NTL == 2 ? NTL * kImg * 8 : 0;
    __shared__ bool run;
    __shared__ __align__(16) char lds[kOverlay + kL + kStage];
    F* const iR = (F*)lds;                             // [tile row][tile column]
    F* const iT = iR + NTL * NTL * kImg;               // [tile column][tile row]
    double* const iS = (double*)(lds + (NTL == 4 ? kR : 2 * kR));  // lower tiles
    double* const iL = (double*)(lds + kOverlay);      // tiles below the diagonal of panels p and p + 1
    // one image per wavefront to turn tiles in, before what is there later
    double* const iStage = NTL == 1 ? iS : kRowLds ? (double*)iT : iL;
    double* const iQ = iL + (2 * NTL - 3) * kImg;      // updated diagonal tiles p and p + 1

    FactorDesc P;
    int lvl;
    int64_t kk;
    fetch_item(L, P, lvl, kk);
    double state;  // of *P.info; used only once the loads below are out
    buf_ld(state, block_rsrc(P.info, 8), 0);

    const int lane = threadIdx.x & 63;
    int r = lane & 15, c = lane >> 4;
    int po[4], tp[4];  // image positions of the register form and of its transpose
    auto positions = [&]() {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            po[v] = img_pos(r, 4 * v + c);
            tp[v] = img_pos(4 * v + c, r);
        }
    };
    positions();
    const int w = NTL == 1 ? 0 : wave_id();
    const int64_t N = P.N;
    const int n = P.n;
    const size_t nn = (size_t)n * n;
    const int64_t s = (int64_t)1 << lvl;
    const int64_t h = s >> 1;
    const int64_t i = (kk * 2 + 1) << lvl;
    const bool has_r = i + s <= N;
    const bool has_l = i > s;
    const bool def_self = lvl > 0 && i + h <= N;
    const bool def_sep = lvl > 0 && has_r && i + 3 * h <= N;
    const int64_t pi = perm_pos(N, lvl, i);
    const int64_t pr = has_r ? perm_pos(N, level_of(i + s), i + s) : 0;
    F *Lf, *Rf, *Tf;
    if constexpr (MODE == 0) {
        Lf = P.Ld;
        Rf = P.Rb;
        Tf = P.Tb;
    } else {
        Lf = P.L32;
        Rf = P.R32;
        Tf = P.T32;
    }
    // a block's resource; nothing is read or written without `on`
    auto rsrc = [&](const auto* p, bool on) { return block_rsrc(p, on ? n * n * (int)sizeof(*p) : 0); };

    // pair d of this wavefront: the other tile row, and whether there is one
    auto other = [&](int d) { return d == 0 ? w : (w + d) % NTL; };
    auto pair_on = [&](int d) {
        return 2 * d < NTL || (2 * d == NTL && w < NTL / 2);
    };
    // Register v of pair d's accumulator is an element of tile (y, w) of S_i or
    // S_{i+s}, y = other(d), always one of the lower triangle's tile (ta, tb):
    // row q(v), column r of it, q(v) = PR::row(v, c), or where y < w (across())
    // row r, column q(v).  As byte offsets: a lane part for v = 0 (at(); also
    // for v when d = 0, whose tile is on the diagonal), plus v times step().
    // Rows past n are past the block's end or masked.
    constexpr int kStep = MODE == 0 ? 4 : 1;
    auto across = [&](int d) { return other(d) < w; };
    auto at = [&](int d, int v) {
        const int y = other(d), q = PR::row(v, c);
        const bool t = across(d);
        const int row = kT * (t ? w : y) + (t ? r : q - kStep * v), col = kT * (t ? y : w) + (t ? q - kStep * v : r);
        return elem_off<double>(row, col, n, pair_on(d) && (!t || row < n) && (d > 0 || r <= q));
    };
    auto step = [&](int d) { return kStep * (across(d) ? 1 : n) * 8; };
    auto load_pair = [&](d4& x, int d, __amdgpu_buffer_rsrc_t rs) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double e;
            buf_ld(e, rs, at(d, v), v * step(d));
            x[v] = e;
        }
    };
    // tile column b of a block as product operand: element (16p + 4v + l/16, 16b + l%16)
    // (rows past n are past the block's end)
    auto load_cols = [&](auto (&x)[NTL][4], int b, __amdgpu_buffer_rsrc_t rs, bool on) {
        using C = std::remove_reference_t<decltype(x[0][0])>;
        const int at = elem_off<C>(c, kT * b + r, n, on && kT * b + r < n);
#pragma unroll
        for (int p = 0; p < NTL; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) buf_ld(x[p][v], rs, at, (kT * p + 4 * v) * n * (int)sizeof(C));
    };
    // tile row w of a block, element (16w + 4v + l/16, 16p + l%16)
    auto load_rows = [&](auto (&x)[NTL][4], __amdgpu_buffer_rsrc_t rs) {
        using C = std::remove_reference_t<decltype(x[0][0])>;
        const int at = elem_off<C>(c, r, n, true);
#pragma unroll
        for (int p = 0; p < NTL; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                buf_ld(x[p][v], rs, r < n - kT * p ? at : kOob, ((kT * w + 4 * v) * n + kT * p) * (int)sizeof(C));
    };
    // couplings: tile row w of C_{i+s,i}, tile column w of C_{i,i-s}
    auto load_couplings = [&](auto (&x)[2][NTL][4], const auto* Cr, const auto* Cl) {
        load_rows(x[0], rsrc(Cr, has_r));
        load_cols(x[1], w, rsrc(Cl, has_l), true);
    };
    // the former into the register form, through this wavefront's own image
    auto turn = [&](auto (&x)[NTL][4]) {
        using C = std::remove_reference_t<decltype(x[0][0])>;
        C* const img = (C*)iStage + w * kImg;
#pragma unroll
        for (int p = 0; p < NTL; ++p) {
#pragma unroll
            for (int v = 0; v < 4; ++v) img[tp[v]] = x[p][v];
            wave_lds_sync();
#pragma unroll
            for (int v = 0; v < 4; ++v) x[p][v] = img[po[v]];
            wave_lds_sync();
        }
    };
    // S -= T^T T of the wavefront's pairs, the products summed before they are
    // subtracted (subtracted from S one after the other, each would be rounded
    // to S's magnitude): tile columns own and other(d)
    // (NTL 2: loaded by this wavefront too; NTL 4: from the images of the
    // wavefronts that carry them)
    auto syrk = [&](d4 (&x)[D], const F (&own)[NTL][4], const F (&oth)[NTL][4], const F* img) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (!pair_on(d)) continue;
            Acc acc = {};
#pragma unroll
            for (int p = 0; p < NTL; ++p) {
                F o[4];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    o[v] = d == 0 ? own[p][v] : NTL >= 3 ? img[(other(d) * NTL + p) * kImg + po[v]] : oth[p][v];
                PR::template tile<false>(acc, o, own[p]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) x[d][v] -= (double)acc[v];
        }
    };
    auto put_img = [&](F* img, const F (&x)[NTL][4]) {
#pragma unroll
        for (int p = 0; p < NTL; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) img[(w * NTL + p) * kImg + po[v]] = x[p][v];
    };

    // 1. all loads, then S_i and S_{i+s} with their deferred updates
    d4 X[kRowLds ? 2 : 3][NTL];  // R_i (tile row w), T_i^T (tile column w), L_ii (tile row a)
    d4 sep[D];
    const int a = NTL == 2 ? 1 : w;  // (two tile rows: both wavefronts carry the lower one)
    d4 Q;
    {
        d4 self[D];
        F t1[NTL][4], t2[NTL][4], o1[NTL][4], o2[NTL][4], x[2][NTL][4];
        const int lo = lvl > 0 ? lvl - 1 : 0;
        const auto rs = rsrc(lvl == 0 ? P.A_diag + (size_t)(i - 1) * nn : P.Ld + (size_t)pi * nn, true);
        const auto rp = rsrc(lvl == 0 ? P.A_diag + (size_t)(i + s - 1) * nn : P.Ld + (size_t)pr * nn, has_r);
        const auto r1 = rsrc(Tf + (size_t)perm_pos(N, lo, i + h) * nn, def_self);
        const auto r2 = rsrc(Tf + (size_t)perm_pos(N, lo, i + 3 * h) * nn, def_sep);
#pragma unroll
        for (int d = 0; d < D; ++d) load_pair(self[d], d, rs);
        load_cols(t1, w, r1, true);
        if constexpr (NTL == 2) load_cols(o1, other(1), r1, pair_on(1));
        if constexpr (MODE == 0) {
            load_couplings(x, lvl == 0 ? P.A_off + (size_t)(i - 1) * nn : Rf + (size_t)pi * nn,
                           lvl == 0 ? P.A_off + (size_t)(i - 2) * nn : Tf + (size_t)pi * nn);
        } else if (lvl > 0) {
            load_couplings(x, (const F*)Rf + (size_t)pi * nn, (const F*)Tf + (size_t)pi * nn);
        } else {
            double y[2][NTL][4];  // the FP64 input blocks
            load_couplings(y, P.A_off + (size_t)(i - 1) * nn, P.A_off + (size_t)(i - 2) * nn);
            turn(y[0]);
#pragma unroll
            for (int p = 0; p < NTL; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    X[0][p][v] = y[0][p][v];
                    X[1][p][v] = y[1][p][v];
                }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) load_pair(sep[d], d, rp);
        if constexpr (NTL < 3) load_cols(t2, w, r2, true);
        if constexpr (NTL == 2) load_cols(o2, other(1), r2, pair_on(1));
        __builtin_amdgcn_sched_barrier(0);

        if (def_self) {
            if constexpr (NTL >= 3) {
                put_img(iR, t1);
                __syncthreads();
            }
            syrk(self, t1, o1, iR);
        }
        if constexpr (NTL >= 3) load_cols(t2, w, r2, true);  // (registers of T')
        if (MODE == 0 || lvl > 0) turn(x[0]);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (!pair_on(d)) continue;
            const int y = other(d), ta = w > y ? w : y, tb = w + y - ta;
            double* const img = iS + (ta * (ta + 1) / 2 + tb) * kImg;
            const bool t = across(d);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int q = PR::row(v, c), row = t ? r : q, col = t ? q : r;
                double e = self[d][v];
                if (d == 0 && row == col && kT * w + row >= n) e = 1.0;
                img[img_pos(row, col)] = e;
            }
        }
        // an earlier level broke down: one wavefront's reading for all of them
        if constexpr (NTL == 1) {
            if (__double_as_longlong(state) != -1) return;
            wave_lds_sync();
        } else {
            if (threadIdx.x == 0) run = __double_as_longlong(state) == -1;
            __syncthreads();
            if (!run) return;
        }
        if (def_sep) {
            if constexpr (NTL >= 3) {
                put_img(iR, t2);  // (T' has been read before the barrier above)
                __syncthreads();
            }
            syrk(sep, t2, o2, iR);
        }
        if (MODE == 0 || lvl > 0) {
#pragma unroll
            for (int p = 0; p < NTL; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    X[0][p][v] = (double)x[0][p][v];
                    X[1][p][v] = (double)x[1][p][v];
                }
        }
    }
    // 2. the panels
    auto load_img = [&](d4& x, const double* img) {
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = img[po[v]];
    };
    load_img(Q, iS);
    if constexpr (!kRowLds) {
#pragma unroll
        for (int b = 0; b < NTL; ++b) {
            X[2][b] = d4{0.0, 0.0, 0.0, 0.0};
            if (NTL > 1 && a > 0 && b <= a) load_img(X[2][b], iS + (a * (a + 1) / 2 + b) * kImg);
        }
    }
    auto tri = [](int x, int y) { return (x * (x + 1) / 2 + y) * kImg; };
    auto store_img = [&](double* img, const d4& x) {
#pragma unroll
        for (int v = 0; v < 4; ++v) img[po[v]] = x[v];
    };
    const int lo = elem_off<F>(c, r, n, true);
    const auto rL = rsrc(Lf + (size_t)pi * nn, true);
    const auto rR = rsrc(Rf + (size_t)pi * nn, has_r), rT = rsrc(Tf + (size_t)pi * nn, has_l);
#pragma unroll (NTL >= 3 ? 1 : NTL)
    for (int p = 0; p < NTL; ++p) {
        d4 E;
#pragma unroll
        for (int v = 0; v < 4; ++v) E[v] = 4 * v + c == r ? 1.0 : 0.0;
        d4 Y[TB];
#pragma unroll
        for (int t = 0; t < (kRowLds ? 2 : TB); ++t) Y[t] = X[t][0];
        if constexpr (kRowLds) {
            Y[2] = d4{0.0, 0.0, 0.0, 0.0};
            if (a > p) load_img(Y[2], iS + tri(a, p));
        }
        bool ok = true;
        const int left = n - kT * p;  // steps past n are the identity
        if (left > 12) {
            // each step's products on the other tiles run under the next
            // step's chain
            const PanelStep s0 = panel_diag<0, MODE == 0>(Q, ok, lane), s1 = panel_diag<1, MODE == 0>(Q, ok, lane);
            panel_rest<TB, 0>(E, Y, s0);
            const PanelStep s2 = panel_diag<2, MODE == 0>(Q, ok, lane);
            panel_rest<TB, 1>(E, Y, s1);
            const PanelStep s3 = panel_diag<3, MODE == 0>(Q, ok, lane);
            panel_rest<TB, 2>(E, Y, s2);
            panel_rest<TB, 3>(E, Y, s3);
        } else {
            panel_rest<TB, 0>(E, Y, panel_diag<0, MODE == 0>(Q, ok, lane));
            if (left > 4) panel_rest<TB, 1>(E, Y, panel_diag<1, MODE == 0>(Q, ok, lane));
            if (left > 8) panel_rest<TB, 2>(E, Y, panel_diag<2, MODE == 0>(Q, ok, lane));
        }
        if (!__builtin_amdgcn_readfirstlane((int)ok)) {  // every wavefront alike
            if (threadIdx.x == 0) atomicMin(P.info, (unsigned long long)i);
            return;
        }
        // stores: a lane part and a part by panel (rows past n are masked by
        // lane or past the block's end); R_i follows from its images.  L_ii
        // below and on the diagonal of a diagonal tile, its inverse transposed
        // above it
        const bool below = NTL > 1 && a > p;
        const int rows = kT * w + r, col = kT * p * (int)sizeof(F);
        const int own = (rows * n + c) * (int)sizeof(F);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            buf_st((F)Y[1][v], rT, rows < n ? lo : kOob, ((kT * p + 4 * v) * n + kT * w) * (int)sizeof(F));
            if (w == p)
                buf_st((F)(r < 4 * v + c ? E[v] : Q[v]), rL, 4 * v + c < left && r < left ? own : kOob,
                       col + 4 * v * (int)sizeof(F));
            if (NTL == 2 && below && w == 1)
                buf_st((F)Y[TB - 1][v], rL, rows < n ? own : kOob, col + 4 * v * (int)sizeof(F));
        }
        X[0][0] = Y[0];
        X[1][0] = Y[1];
        if constexpr (NTL == 1) continue;
        if constexpr (NTL >= 3) {
            if (p + 1 < NTL) {
                double* const img = kRowLds ? iS + tri(a, p) : iL + ((p & 1) * (NTL - 1) + a - 1 - p) * kImg;
                if (below) {
                    store_img(img, Y[TB - 1]);
                    wave_lds_sync();
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        buf_st((F)img[tp[v]], rL, lo, ((kT * w + 4 * v) * n + kT * p) * (int)sizeof(F));
                }
                double* const next = kRowLds ? iS + tri(p + 1, p + 1) : iQ + (p & 1) * kImg;
                if (a == p + 1) {
                    if constexpr (kRowLds) {
                        d4 x;
                        load_img(x, next);
                        sub_abt(x, Y[TB - 1], Y[TB - 1]);
                        store_img(next, x);
                    } else {
                        sub_abt(X[2][1], Y[TB - 1], Y[TB - 1]);
                        store_img(next, X[2][1]);
                    }
                }
                __syncthreads();
                load_img(Q, next);
            }
        }
        // the images for step 3 (from NTL = 3 on in the place of others, which all
        // wavefronts have read before the barrier above)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            iR[(w * NTL + p) * kImg + po[v]] = (F)Y[0][v];
            iT[(w * NTL + p) * kImg + po[v]] = (F)Y[1][v];
        }
#pragma unroll
        for (int q = 1; q < NTL; ++q) {
            if (p + q >= NTL) break;
            d4 lq;
            if constexpr (kRowLds) load_img(lq, iS + tri(p + q, p));
            else if constexpr (NTL >= 3) load_img(lq, iL + ((p & 1) * (NTL - 1) + q - 1) * kImg);
            else lq = Y[TB - 1];
            sub_abt(X[0][q], X[0][0], lq);
            sub_abt(X[1][q], X[1][0], lq);
            if (NTL == 2 || (q > 1 ? p + q <= a : a > p + 1)) {
                if constexpr (kRowLds) {
                    d4 x;
                    load_img(x, iS + tri(a, p + q));
                    sub_abt(x, Y[TB - 1], lq);
                    store_img(iS + tri(a, p + q), x);
                } else {
                    sub_abt(X[2][q], Y[TB - 1], lq);
                }
            }
        }
        if constexpr (NTL == 2) Q = X[2][1];
#pragma unroll
        for (int q = 1; q < NTL; ++q)
#pragma unroll
            for (int t = 0; t < (kRowLds ? 2 : TB); ++t) X[t][q - 1] = X[t][q];
    }
    if (!has_r) return;
    // the addresses of the stores below are formed anew: kept through the panels
    // they leave too few registers there (spills at four tile rows)
    asm volatile("" : "+v"(r), "+v"(c));
    positions();
    if constexpr (NTL > 1) {
        __syncthreads();
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) ((F*)iS)[po[v]] = (F)X[0][0][v];
        wave_lds_sync();
    }
    const F* const img = NTL == 1 ? (const F*)iS : iR + w * NTL * kImg;
#pragma unroll
    for (int p = 0; p < NTL; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            buf_st(img[p * kImg + tp[v]], rR, r < n - kT * p ? lo : kOob,
                   ((kT * w + 4 * v) * n + kT * p) * (int)sizeof(F));

    // 3. separator update and fill
    auto load_op = [&](F (&x)[4], const F* img, const d4& reg) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if constexpr (NTL == 1) x[v] = (F)reg[v];
            else x[v] = img[po[v]];
        }
    };
    const auto rp = rsrc(P.Ld + (size_t)pr * nn, true);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (!pair_on(d)) continue;
        Acc acc = {};
#pragma unroll
        for (int p = 0; p < NTL; ++p) {
            F x[4], y[4];
            load_op(x, iR + (other(d) * NTL + p) * kImg, X[0][0]);
            load_op(y, iR + (w * NTL + p) * kImg, X[0][0]);
            PR::template tile<false>(acc, x, y);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) buf_st(sep[d][v] - (double)acc[v], rp, at(d, v), v * step(d));
    }
    if (!has_l) return;
    Acc f[NTL];
#pragma unroll
    for (int b = 0; b < NTL; ++b) f[b] = Acc{};
#pragma unroll
    for (int p = 0; p < NTL; ++p) {
        F y[4];
        load_op(y, iT + (w * NTL + p) * kImg, X[1][0]);
#pragma unroll
        for (int b = 0; b < NTL; ++b) {
            F x[4];
            load_op(x, iR + (b * NTL + p) * kImg, X[0][0]);
            PR::template tile<true>(f[b], x, y);
        }
    }
    const int64_t lft = i - s, rgt = i + s;
    const auto rf = rsrc((((lft >> (lvl + 1)) & 1) != 0) ? Rf + (size_t)perm_pos(N, lvl + 1, lft) * nn
                                                         : Tf + (size_t)perm_pos(N, lvl + 1, rgt) * nn,
                         true);
    const int fo = elem_off<F>(PR::row(0, c), kT * w + r, n, kT * w + r < n);
#pragma unroll
    for (int b = 0; b < NTL; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) buf_st(f[b][v], rf, fo, (kT * b + kStep * v) * n * (int)sizeof(F));
}

// One launch over the nodes of a level, padded size np <= 64.
template <int MODE>
hipError_t launch_factor_node(const Launch<FactorDesc>& p, int np, int64_t items, hipStream_t st) {
    const dim3 g((unsigned)items);
    switch (np) {
        case 8:
        case 16: hipLaunchKernelGGL((k_factor_node<1, MODE>), g, dim3(kWave), 0, st, p); break;
        case 32: hipLaunchKernelGGL((k_factor_node<2, MODE>), g, dim3(2 * kWave), 0, st, p); break;
        case 48: hipLaunchKernelGGL((k_factor_node<3, MODE>), g, dim3(3 * kWave), 0, st, p); break;
        case 64: hipLaunchKernelGGL((k_factor_node<4, MODE>), g, dim3(4 * kWave), 0, st, p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace node
}  // namespace btc
