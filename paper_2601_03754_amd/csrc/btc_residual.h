// FP64 residual b - Psi x, every n x n block read from HBM once.
//
//   block row i: r_i = b_i - D_i x_i - E_{i-1} x_{i-1} - E_i^T x_{i+1}
//
// Two launches.  The workgroup of block row i reads the lower triangle of D_i
// and E_i (block (i+1, i)), wavefront w the tiles of tile row w, and uses
// every tile twice:
//   P_i     = b_i - D_i x_i - E_i^T x_{i+1}
//   Q_{i+1} = E_i x_i
// the second launch forms r_i = P_i - Q_i, its copies and the per-column
// partial squared norms of r_i and b_i.
//
// All loads of a wavefront go out before the first product, four rows of 16
// elements each: register v of lane l holds element (4v + l/16, l%16) of a
// tile M.  That is the A operand of v_mfma_f64_4x4x4 for M^T (the lanes of one
// of its four 4 x 4 blocks hold four rows of M^T), so M^T x takes four of them
// per four columns of x; M x takes one fma per register and column, and only
// the sum over a tile row is added up over its 16 lanes, once per row block
// and not per tile.  What bounds it is memory; it took the place of a form
// with one wavefront per block row and a sum over the wavefront for every row
// of every block.  Measured, first launch, before -> after: N = 4096, n = 64,
// m = 4: 167 -> 65 us (memory floor 40); n = 96, m = 4: 500 -> 116, m = 1: 106 ->
// 98 (floor 91); n = 128, m = 1: 167 -> 171; N = 20 000, n = 32, m = 4: 373 -> 86;
// N = 511, n = 50, m = 1: 16.3 -> 6.8.
#pragma once

#include "btc_device.h"
#include "btc_kernels.h"

namespace btc {
namespace {

// Value of the exchange partner across lane bit H of a row of 16 lanes (DPP:
// the row mirror for bit 3, the half-row mirror for bit 2, quad permutations
// for bits 1 and 0).  Each pairing is an involution whose pairs differ in bit H
// and otherwise only in lower bits.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const long long w = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)w, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(w >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int H>
__device__ __forceinline__ double partner(double v) {
    if constexpr (H == 8) return dpp_d<0x140>(v);       // row_mirror
    else if constexpr (H == 4) return dpp_d<0x141>(v);  // row_half_mirror
    else if constexpr (H == 2) return dpp_d<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    else return dpp_d<0xB1>(v);                         // quad_perm [1, 0, 3, 2]
}
// Lane bit of exchange step T: bits 3, 2, 1, 0 (a mirror also flips the bits
// below its own, so those must not be bound to a value yet).
constexpr int step_bit(int t) { return 8 >> t; }

// Halving exchanges from step T on, W values per lane in play: the lane
// keeps the half its step bit selects and adds its partner's copy of it.
template <int W, int T>
__device__ __forceinline__ void halve(double* v, int lane) {
    if constexpr (W >= 1) {
        constexpr int H = step_bit(T);
        const bool up = (lane & H) != 0;
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const double send = up ? v[j] : v[j + W];
            const double keep = up ? v[j + W] : v[j];
            v[j] = keep + partner<H>(send);
        }
        halve<W / 2, T + 1>(v, lane);
    }
}
// Sum over rows of 16 lanes of KB values per lane (4 or 16): lane r of a row is
// left with the total of value r (KB 16) or r / 4 (KB 4).  Every total is
// formed by the same tree of additions whatever KB is.
template <int KB>
__device__ __forceinline__ double row_sums(double (&v)[KB], int lane) {
    static_assert(KB == 4 || KB == 16, "values per lane");
    halve<KB / 2, 0>(v, lane);
    double s = v[0];
    if constexpr (KB == 4) {
        s += partner<2>(s);
        s += partner<1>(s);
    }
    return s;
}

// Wavefronts of a workgroup: one per tile row, or (from six tile rows on, where
// two blocks' tiles do not fit the registers beside the sums) one per two of
// them, w and NTL - 1 - w, a block at a time.
template <int NTL>
constexpr int res_rows() { return NTL >= 6 ? 2 : 1; }

// MC: right-hand-side columns per pass over the tiles (1 or 4; the same
// arithmetic for a column either way).  In the results' lane layout lane l
// holds row 4 ((l%16) / 4) + l/16 of a tile, column l % 4 of the pass.
template <int NTL, int MC>
__global__ __launch_bounds__(NTL / res_rows<NTL>() * kWave, NTL >= 6 ? (MC == 1 ? 3 : 2) : 1) void k_res(
    Launch<ResidualDesc> L) {
    constexpr int kT = 16, RW = res_rows<NTL>(), W = NTL / RW;
    __shared__ double xs[NTL * kT][MC];      // x_i of the pass
    __shared__ double red[W][NTL][kWave];    // [wavefront][tile row]: its share of D_i x_i + E_i^T x_{i+1}
    ResidualDesc P;
    int64_t row0;
    {
        const unsigned b = xcd_local_block();
        if (L.items) {
            const WorkItem it = L.items[b];
            P = L.descs[it.inst];
            row0 = it.k;
        } else {
            P = L.single;
            row0 = b;
        }
    }
    if (P.state && P.state->done) return;
    const int lane = threadIdx.x & 63, r = lane & 15, c = lane >> 4;
    const int w = W == 1 ? 0 : wave_id();
    const int64_t N = P.N;
    const int n = P.n, m = P.m;
    const size_t nn = (size_t)n * n, nm = (size_t)n * m;
    const int64_t i = row0 + 1;
    const bool rgt = i < N;
    const double* const x1 = P.X + (size_t)(i - 1) * nm;
    const double* const x2 = P.X + (size_t)(rgt ? i : i - 1) * nm;

    // element (row, column q) of a block of vectors, 0 outside (and unless on)
    auto vec = [&](const double* x, int row, int q, bool on) {
        const bool ok = on && row < n && q < m;
        const double v = x[ok ? (size_t)row * m + q : 0];
        return ok ? v : 0.0;
    };
    static_assert(W * kWave >= NTL * kT, "a thread per row");
    const int row = threadIdx.x;
    double xn[MC], xw[4], xr[4];
    // x_i for all wavefronts
    auto fetch_x = [&](int q0) {
#pragma unroll
        for (int j = 0; j < MC; ++j) xn[j] = vec(x1, row, q0 + j, row < NTL * kT);
    };
    // x_i and x_{i+1} of tile row a as B operands
    auto fetch_row = [&](int a, int q0) {
        const int j = lane & 3;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            xw[v] = vec(x1, kT * a + 4 * v + c, q0 + j, j < MC);
            xr[v] = vec(x2, kT * a + 4 * v + c, q0 + j, j < MC && rgt);
        }
    };
    const auto re = block_rsrc(P.A_off + (size_t)(i - 1) * nn, rgt ? n * n * 8 : 0);
    const auto rd = block_rsrc(P.A_diag + (size_t)(i - 1) * nn, n * n * 8);
    const int lo = elem_off<double>(c, r, n, true);  // rows past n are past the block's end
    auto load_tiles = [&](double (&M)[NTL][4], int a, bool lower) {
#pragma unroll
        for (int b = 0; b < NTL; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                buf_ld(M[b][v], lower ? rd : re,
                       (!lower || kT * b + r <= kT * a + 4 * v + c) && r < n - kT * b ? lo : kOob,
                       ((kT * a + 4 * v) * n + kT * b) * 8);
    };
    fetch_x(0);
    double e[NTL][4], d[RW == 1 ? NTL : 1][4];
    if constexpr (RW == 1) {
        fetch_row(w, 0);
        load_tiles(e, w, false);
        load_tiles(d, w, true);
    }

    for (int q0 = 0; q0 < m; q0 += MC) {
        if (row < NTL * kT)
#pragma unroll
            for (int j = 0; j < MC; ++j) xs[row][j] = xn[j];
        __syncthreads();
        double cr[NTL];
#pragma unroll
        for (int b = 0; b < NTL; ++b) cr[b] = 0.0;
        const int q = q0 + (r & 3), rr = 4 * (r >> 2) + c;  // this lane's column, row of a tile
        const bool mine = (MC == 4 || (r & 3) == 0) && q < m;
        // a block's tile row a: its part of M x (returned), M^T x into cr
        auto block = [&](const double (&M)[NTL][4], const double (&x)[4], int a, bool lower) {
            double s[4 * MC];
#pragma unroll
            for (int k = 0; k < 4 * MC; ++k) s[k] = 0.0;
#pragma unroll
            for (int b = 0; b < NTL; ++b) {
                if (lower && b > a) break;
                double y[MC];
#pragma unroll
                for (int j = 0; j < MC; ++j) y[j] = xs[kT * b + r][j];
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int j = 0; j < MC; ++j) s[v * MC + j] = fma(M[b][v], y[j], s[v * MC + j]);
                // (the diagonal of D_i counts once)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    cr[b] = __builtin_amdgcn_mfma_f64_4x4x4f64(lower && b == a && r == 4 * v + c ? 0.0 : M[b][v], x[v],
                                                               cr[b], 0, 0, 0);
            }
            return row_sums(s, lane);
        };
        auto add_own = [&](int a, double t) {
#pragma unroll
            for (int b = 0; b < NTL; ++b)
                if (b == a) cr[b] += t;
        };
        auto store_q = [&](int a, double t) {
            if (mine && kT * a + rr < n) P.Q[(size_t)i * nm + (size_t)(kT * a + rr) * m + q] = t;
        };
        if constexpr (RW == 1) {
            if (rgt) store_q(w, block(e, xr, w, false));
            add_own(w, block(d, xw, w, true));
            if (q0 + MC < m) fetch_row(w, q0 + MC);
        } else {
#pragma unroll 1
            for (int h = 0; h < RW; ++h) {
                const int a = h ? NTL - 1 - w : w;
                fetch_row(a, q0);
                if (rgt) {
                    load_tiles(e, a, false);
                    store_q(a, block(e, xr, a, false));
                }
                load_tiles(e, a, true);
                add_own(a, block(e, xw, a, true));
            }
        }
        if (q0 + MC < m) fetch_x(q0 + MC);
#pragma unroll
        for (int b = 0; b < NTL; ++b) red[w][b][lane] = cr[b];
        __syncthreads();
#pragma unroll
        for (int h = 0; h < RW; ++h) {
            const int a = h ? NTL - 1 - w : w;
            double sum = red[0][a][lane];
#pragma unroll
            for (int k = 1; k < W; ++k) sum += red[k][a][lane];
            const size_t at = (size_t)(i - 1) * nm + (size_t)(kT * a + rr) * m + q;
            if (mine && kT * a + rr < n) P.P[at] = P.B[at] - sum;
        }
    }
}

// r_i = P_i - Q_i (Q_1 = 0), its FP32 copy and the partial norms; one
// wavefront per block row, four to a workgroup, MC columns at a time.
constexpr int kFinRows = 4;
template <int MC>
__global__ __launch_bounds__(kFinRows * kWave) void k_res_fin(Launch<ResidualDesc> L, int64_t items) {
    const int64_t idx = (int64_t)blockIdx.x * kFinRows + wave_id();
    if (idx >= items) return;
    ResidualDesc P;
    int level;
    int64_t row0;
    fetch_item_at(L, idx, P, level, row0);
    if (P.state && P.state->done) return;
    const int lane = threadIdx.x & 63;
    const int n = P.n, m = P.m;
    const int64_t i = row0 + 1;
    const size_t base = (size_t)(i - 1) * n * m;
    for (int q0 = 0; q0 < m; q0 += MC) {
        double r2[MC] = {}, b2[MC] = {};
        for (int r = lane; r < n; r += kWave) {
            double p[MC], q[MC], b[MC];
#pragma unroll
            for (int j = 0; j < MC; ++j) {
                const size_t e = base + (size_t)r * m + (q0 + j < m ? q0 + j : q0);
                p[j] = P.P[e];
                q[j] = i > 1 ? P.Q[e] : 0.0;
                b[j] = P.B[e];
            }
#pragma unroll
            for (int j = 0; j < MC; ++j) {
                if (q0 + j >= m) break;
                const size_t e = base + (size_t)r * m + q0 + j;
                const double v = p[j] - q[j];
                if (P.R32) P.R32[e] = (float)v;
                if (P.R64) P.R64[e] = P.neg ? -v : v;
                r2[j] = fma(v, v, r2[j]);
                b2[j] = fma(b[j], b[j], b2[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < MC; ++j) {
            if (q0 + j >= m) break;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                r2[j] += __shfl_xor(r2[j], off);
                b2[j] += __shfl_xor(b2[j], off);
            }
            if (lane == 0) {
                P.part[((size_t)(i - 1) * m + q0 + j) * 2 + 0] = r2[j];
                P.part[((size_t)(i - 1) * m + q0 + j) * 2 + 1] = b2[j];
            }
        }
    }
}

template <int NTL, int MC>
hipError_t launch_res_mc(const Launch<ResidualDesc>& p, int64_t items, hipStream_t st) {
    hipLaunchKernelGGL((k_res<NTL, MC>), dim3((unsigned)items), dim3(NTL / res_rows<NTL>() * kWave), 0, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_res_fin<MC>, dim3((unsigned)((items + kFinRows - 1) / kFinRows)), dim3(kFinRows * kWave), 0, st,
                       p, items);
    return hipGetLastError();
}
template <int NTL>
hipError_t launch_res_np(const Launch<ResidualDesc>& p, int64_t items, int mc, hipStream_t st) {
    return mc <= 1 ? launch_res_mc<NTL, 1>(p, items, st) : launch_res_mc<NTL, 4>(p, items, st);
}

}  // namespace

hipError_t launch_residual(const Launch<ResidualDesc>& p, int np, int64_t items, int mc, hipStream_t st) {
    switch (np) {
        case 8:
        case 16: return launch_res_np<1>(p, items, mc, st);
        case 32: return launch_res_np<2>(p, items, mc, st);
        case 48: return launch_res_np<3>(p, items, mc, st);
        case 64: return launch_res_np<4>(p, items, mc, st);
        case 80:
        case 96: return launch_res_np<6>(p, items, mc, st);
        case 128: return launch_res_np<8>(p, items, mc, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace btc
