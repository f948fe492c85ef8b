// Matrix-core tile helpers shared by the factorization kernels (gfx950).
//
// Blocks are staged in LDS padded to NP x NP with an odd row stride and split
// into 16 x 16 tiles; block products run on MFMA instructions whose operand
// and accumulator lane layouts are:
//   v_mfma_f64_16x16x4f64 : A[i][k] in lane i + 16k, B[k][j] in lane j + 16k,
//                           accumulator register v of lane l = element
//                           (4v + l/16, l%16)
//   v_mfma_f32_16x16x4f32 : same operand layout (one float per lane),
//                           accumulator register v of lane l = element
//                           (4(l/16) + v, l%16)
#pragma once

#include "btc_device.h"
#include "btc_failword.h"

namespace btc {
namespace tiles {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kT = 16;       // tile side
constexpr int kLDI = kT + 1; // row stride of an inverted diagonal tile in LDS

// f64 16x16x4 accumulator layout: register v of lane l holds tile element
// (4v + l/16, l%16).  Operand layouts: A[i][k] in lane i + 16k, B[k][j] in
// lane j + 16k.
__device__ __forceinline__ int acc_r(int v, int lane) { return 4 * v + (lane >> 4); }
__device__ __forceinline__ int acc_c(int lane) { return lane & 15; }

// acc += (NEG ? -1 : 1) * sum_{kk<K} opA[ra+i][ka+kk] * opB[kb+kk][cb+j]
//   opA[r][k] = TA ? A[k][r] : A[r][k],  opB[k][c] = TB ? B[c][k] : B[k][c]
template <int LDA, int LDB, bool TA, bool TB, bool NEG>
__device__ __forceinline__ void mma_tile(d4& acc, const double* __restrict__ A, int ra, int ka,
                                         const double* __restrict__ B, int cb, int kb, int K) {
    const int lane = threadIdx.x & 63;
    const int i = lane & 15, q = lane >> 4;
    auto opa = [&](int kk) {
        const int k1 = ka + kk + q;
        const double a = TA ? A[k1 * LDA + ra + i] : A[(ra + i) * LDA + k1];
        return NEG ? -a : a;
    };
    auto opb = [&](int kk) {
        const int k2 = kb + kk + q;
        return TB ? B[(cb + i) * LDB + k2] : B[k2 * LDB + cb + i];
    };
    if (K >= 16 && K % 8 == 0) {
        // two independent accumulation chains (hides the matrix-core latency)
        d4 acc1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
        for (int kk = 0; kk < K; kk += 8) {
            const double a0 = opa(kk), b0 = opb(kk), a1 = opa(kk + 4), b1 = opb(kk + 4);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc1, 0, 0, 0);
        }
        acc += acc1;
        return;
    }
#pragma unroll 4
    for (int kk = 0; kk < K; kk += 4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(opa(kk), opb(kk), acc, 0, 0, 0);
}

template <int LD>
__device__ __forceinline__ void acc_load_lds(d4& acc, const double* __restrict__ S, int r0, int c0) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = S[(r0 + acc_r(v, lane)) * LD + c0 + acc_c(lane)];
}

template <int LD>
__device__ __forceinline__ void acc_store_lds(const d4& acc, double* __restrict__ S, int r0, int c0) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v) S[(r0 + acc_r(v, lane)) * LD + c0 + acc_c(lane)] = acc[v];
}

// LDS layout of the lower triangle of an NP x NP block: its 16 x 16 tiles
// (a, b), b <= a, at position a(a+1)/2 + b, rows of kLDI elements (conflict-free
// 16 x 4 operand reads).
struct PackedLds {
    static constexpr int LDT = kLDI;
    static constexpr int kTile = kT * kLDI;
    template <class T>
    __device__ static T* tile(T* A, int a, int b) { return A + (a * (a + 1) / 2 + b) * kTile; }
};
template <int NP>
constexpr int packed_lds_elems() { return (NP / kT) * (NP / kT + 1) / 2 * PackedLds::kTile; }

// k-th lower-triangle tile (a, b), b <= a, in row-major order of the triangle.
__device__ __forceinline__ void tri_tile(int k, int& a, int& b) {
    a = 0;
    while ((a + 1) * (a + 2) / 2 <= k) ++a;
    b = k - a * (a + 1) / 2;
}

// 1/sqrt(p): hardware estimate r refined by one third-order step.  With
// e = 1 - p r^2, 1/sqrt(p) = r (1 - e)^(-1/2) = r (1 + e/2 + 3e^2/8 + ...);
// the estimate's e of about 1e-7 leaves a truncation term near 1e-22, and
// the chain is four dependent operations instead of two Newton steps' six.
__device__ __forceinline__ double rsqrt_refined(double p) {
    const double r = __builtin_amdgcn_rsq(p);
    const double e = fma(-p * r, r, 1.0);
    return fma(r * e, fma(e, 0.375, 0.5), r);
}

// Quad JB of every row of 16 lanes to all four quads of that row.
template <int CTRL, int BANK>
__device__ __forceinline__ double dpp_bank(double old, double x) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(x), CTRL, 0xF, BANK, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(x), CTRL, 0xF, BANK, false);
    return __hiloint2double(hi, lo);
}
template <int JB>
__device__ __forceinline__ double quad_bcast(double x) {
    // quad b takes quad JB: a rotation by 4 (b - JB) lanes (row_ror)
    double y = dpp_bank<0x124, 1 << ((JB + 1) & 3)>(x, x);
    y = dpp_bank<0x128, 1 << ((JB + 2) & 3)>(y, x);
    return dpp_bank<0x12C, 1 << ((JB + 3) & 3)>(y, x);
}

__device__ __forceinline__ double mma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// A 16 x 16 tile in four registers: register jb of lane l holds element (row
// l % 16, column 4 jb + l / 16).  That is both the B operand (4 x 16, its
// transpose) and the accumulator layout of v_mfma_f64_4x4x4 with four blocks,
// so the products below chain through registers with no data movement; their
// A operand, a 4 x 4 block in all four blocks (lane i + 4b + 16k: element
// (i, k)), is a quad broadcast.
//
// Panel step KB: the 4 x 4 diagonal block of the panel's diagonal tile, its
// Cholesky factor and the inverse M of that on every lane alike (ten values
// by readlane; the only serial chain: four reciprocal square roots), then for
// every tile of the panel X = (column block KB) M^T and the rank-4 update of
// the column blocks right of it.  The same products applied to the identity
// (E, register a of lane l: element (4a + l / 16, l % 16)) leave the inverse
// of the diagonal tile.  The chain it replaces held one row per lane and
// broadcast every multiplier by readlane (16 steps of about 300 cycles a
// panel), with the diagonal tiles inverted at the end.  Measured, one node of
// n = 96 alone in its launch: k_tiled_potrf_trsm 35.5 -> 29.6 us in FP64 (28.4
// before it kept the block's own rows, OWN below); of n = 128 52.7 (49.9).
// (panel_diag is the chain, panel_rest what hangs on it.)
struct PanelStep {
    double m;   // lane i + 4b + 16k: M[i][k]
    double y1, y2, y3;  // minus the factored column's blocks below the diagonal, as A operands
};
// OWN: the block's own rows are the factor as computed.  Q M^T repeats them with
// an error that grows with the block's condition, which the sweeps' tile inverse
// does not share; a factor that is rounded to FP32 hides it up to a condition of
// 5e8, beyond what its FP32 Schur products stand, and goes without (18 selects a
// step: 2% of the factorization at n = 50).
template <int KB, bool OWN, class V>
__device__ __forceinline__ PanelStep panel_diag(V& Q, bool& ok, int lane) {
    const int r = lane & 15, c = lane >> 4, i = lane & 3;
    const double q = Q[KB];
    const double d00 = readlane_d(q, 4 * KB), d10 = readlane_d(q, 4 * KB + 1), d20 = readlane_d(q, 4 * KB + 2),
                 d30 = readlane_d(q, 4 * KB + 3), d11 = readlane_d(q, 4 * KB + 17), d21 = readlane_d(q, 4 * KB + 18),
                 d31 = readlane_d(q, 4 * KB + 19), d22 = readlane_d(q, 4 * KB + 34), d32 = readlane_d(q, 4 * KB + 35),
                 d33 = readlane_d(q, 4 * KB + 51);
    const double r0 = rsqrt_refined(d00);
    const double l10 = d10 * r0, l20 = d20 * r0, l30 = d30 * r0;
    const double p1 = fma(-l10, l10, d11), r1 = rsqrt_refined(p1);
    const double l21 = fma(-l20, l10, d21) * r1, l31 = fma(-l30, l10, d31) * r1;
    const double p2 = fma(-l21, l21, fma(-l20, l20, d22)), r2 = rsqrt_refined(p2);
    const double l32 = fma(-l31, l21, fma(-l30, l20, d32)) * r2;
    const double p3 = fma(-l32, l32, fma(-l31, l31, fma(-l30, l30, d33))), r3 = rsqrt_refined(p3);
    ok = ok && d00 > 0.0 && p1 > 0.0 && p2 > 0.0 && p3 > 0.0;
    // column c of M by forward substitution, then row i of it
    const double x0 = c == 0 ? r0 : 0.0;
    const double x1 = fma(-l10, x0, c == 1 ? 1.0 : 0.0) * r1;
    const double x2 = fma(-l21, x1, fma(-l20, x0, c == 2 ? 1.0 : 0.0)) * r2;
    const double x3 = fma(-l32, x2, fma(-l31, x1, fma(-l30, x0, c == 3 ? 1.0 : 0.0))) * r3;
    PanelStep s{};
    s.m = i == 0 ? x0 : i == 1 ? x1 : i == 2 ? x2 : x3;
    const double xq = mma4(s.m, q, 0.0);
    double x = r >= 4 * KB + c ? xq : 0.0;
    if constexpr (OWN) {
        const double l0 = i == 0 ? d00 * r0 : i == 1 ? l10 : i == 2 ? l20 : l30;
        const double l1 = i == 1 ? p1 * r1 : i == 2 ? l21 : l31;
        const double l2 = i == 2 ? p2 * r2 : l32;
        const double own = c == 0 ? l0 : c == 1 ? l1 : c == 2 ? l2 : p3 * r3;
        x = (r >> 2) == KB ? own : xq;
    }
    Q[KB] = x;
    if constexpr (KB < 3) {
        // the next diagonal block first
        s.y1 = -quad_bcast<(KB + 1) & 3>(x);
        Q[KB + 1] = mma4(s.y1, x, Q[KB + 1]);
    }
    if constexpr (KB < 2) {
        s.y2 = -quad_bcast<(KB + 2) & 3>(x);
        Q[KB + 2] = mma4(s.y2, x, Q[KB + 2]);
    }
    if constexpr (KB < 1) {
        s.y3 = -quad_bcast<3>(x);
        Q[3] = mma4(s.y3, x, Q[3]);
    }
    return s;
}
template <int KB, class V>
__device__ __forceinline__ void panel_apply(V& t, const PanelStep& s) {
    const double z = mma4(s.m, t[KB], 0.0);
    t[KB] = z;
    if constexpr (KB < 3) t[KB + 1] = mma4(s.y1, z, t[KB + 1]);
    if constexpr (KB < 2) t[KB + 2] = mma4(s.y2, z, t[KB + 2]);
    if constexpr (KB < 1) t[3] = mma4(s.y3, z, t[3]);
}
template <int TB, int KB, class V>
__device__ __forceinline__ void panel_rest(V& E, V (&S)[TB], const PanelStep& s) {
    panel_apply<KB>(E, s);
#pragma unroll
    for (int t = 0; t < TB; ++t) panel_apply<KB>(S[t], s);
}
// Blocked Cholesky of the lower triangle of an NP x NP LDS block by all NW
// wavefronts of the workgroup (every thread must call it), in 16-column
// panels.  Each panel wavefront holds the diagonal tile (every one repeats
// its steps, so no wavefront waits on another inside a panel) and up to TB
// tiles below it.  Look-ahead: the panel wavefronts of panel p+1 apply panel
// p's update to their own tiles of column p+1 (A_ap -= L_ap L_(p+1)p^T, read
// from LDS straight into the panel's register layout) and factor it at once,
// while the other wavefronts update the trailing tiles right of column p+1.
// The factored diagonal tile and its inverse stay in wavefront 0's registers
// until the barrier (the other panel wavefronts read the unfactored tile).
// On return: L in the lower triangle (tiles above the diagonal untouched),
// 1/L_jj in invd, the inverse of each diagonal tile transposed in its strict
// upper part.  *fail (LDS, 0 on entry) becomes the mark of the first panel with a
// non-positive or NaN pivot; the result is then false for every thread, after the
// same barrier.
// OWN: as in panel_diag.
template <int NP, int NW, bool OWN>
__device__ __forceinline__ bool potrf_blocked(double* __restrict__ A, double* __restrict__ invd, int* fail) {
    using Lay = PackedLds;
    constexpr int NTL = NP / kT;
    constexpr int LT = Lay::LDT;
    // tiles below the diagonal tile per panel wavefront (one where that leaves
    // wavefronts for the trailing update, and at n = 64, whose register budget
    // holds no second one)
    constexpr int TB = NTL <= 4 || NW >= 2 * (NTL - 1) ? 1 : 2;
    // wavefronts that factor panel q
    constexpr auto pwaves = [](int q) { return NTL - 1 - q <= 0 ? 1 : (NTL - 1 - q + TB - 1) / TB; };
    static_assert(pwaves(0) <= NW, "too few wavefronts for the first panel");
    static_assert(NTL <= 2 || pwaves(1) < NW, "the trailing update needs a wavefront outside the panel");
    const int tid = threadIdx.x;
    const int w = wave_id();
    const int lane = tid & 63;
    const int r = lane & 15, c = lane >> 4;
    double Q[4], E[4], S[TB][4];
    auto load_tile = [&](double (&t)[4], const double* T) {
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = T[r * LT + 4 * j + c];
    };
    // factor panel q (tiles in Q and S): the rows below and 1/L_jj to LDS
    auto factor = [&](int q) {
        bool ok = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) E[j] = 4 * j + c == r ? 1.0 : 0.0;
        panel_rest<TB, 0>(E, S, panel_diag<0, OWN>(Q, ok, lane));
        panel_rest<TB, 1>(E, S, panel_diag<1, OWN>(Q, ok, lane));
        panel_rest<TB, 2>(E, S, panel_diag<2, OWN>(Q, ok, lane));
        panel_rest<TB, 3>(E, S, panel_diag<3, OWN>(Q, ok, lane));
        if (!ok && lane == 0) __hip_atomic_store(fail, panel_mark(q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int ta = q + 1 + TB * w + t;
            if (ta >= NTL) break;
            double* T = Lay::tile(A, ta, q);
#pragma unroll
            for (int j = 0; j < 4; ++j) T[r * LT + 4 * j + c] = S[t][j];
        }
        // the inverse's diagonal
        if (w == 0 && c == (r & 3)) invd[q * kT + r] = r < 4 ? E[0] : r < 8 ? E[1] : r < 12 ? E[2] : E[3];
    };
    // wavefront 0's factored diagonal tile q and its inverse into place
    auto place_diag = [&](int q) {
        if (w != 0) return;
        double* T = Lay::tile(A, q, q);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            T[r * LT + 4 * j + c] = r < 4 * j + c ? E[j] : Q[j];
        }
    };
    // A_ab -= L_ap L_bp^T
    auto update = [&](int ta, int tb, int p) {
        double* Tab = Lay::tile(A, ta, tb);
        d4 acc;
        acc_load_lds<LT>(acc, Tab, 0, 0);
        mma_tile<LT, LT, false, true, true>(acc, Lay::tile(A, ta, p), 0, 0, Lay::tile(A, tb, p), 0, 0, kT);
        acc_store_lds<LT>(acc, Tab, 0, 0);
    };
    // (after panel q's barrier)
    auto broke_down = [&](int q) {
        return panel_failed(__hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP), q);
    };
    if (w < pwaves(0)) {
        load_tile(Q, Lay::tile(A, 0, 0));
#pragma unroll
        for (int t = 0; t < TB; ++t)
            if (1 + TB * w + t < NTL) load_tile(S[t], Lay::tile(A, 1 + TB * w + t, 0));
        factor(0);
    }
    __syncthreads();
    if (broke_down(0)) return false;
#pragma unroll 1
    for (int p = 0; p + 1 < NTL; ++p) {
        const int q = p + 1;
        const int pw = pwaves(q);
        place_diag(p);
        if (w < pw) {
            // this wavefront's tiles of column q, minus panel p's share
            double a[4][4];  // -L_qp, column block j, k step s
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int s = 0; s < 4; ++s) a[j][s] = -Lay::tile(A, q, p)[(4 * j + (lane & 3)) * LT + 4 * s + c];
            auto updated = [&](double (&t)[4], int ta) {
                double b[4];
                load_tile(b, Lay::tile(A, ta, p));
                load_tile(t, Lay::tile(A, ta, q));
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j) t[j] = mma4(a[j][s], b[s], t[j]);
            };
            updated(Q, q);
#pragma unroll
            for (int t = 0; t < TB; ++t)
                if (q + 1 + TB * w + t < NTL) updated(S[t], q + 1 + TB * w + t);
            factor(q);
        } else {
            // the trailing tiles right of column q
            const int m = NTL - 1 - q;
            for (int k = w - pw; k < m * (m + 1) / 2; k += NW - pw) {
                int ta, tb;
                tri_tile(k, ta, tb);
                update(q + 1 + ta, q + 1 + tb, p);
            }
        }
        __syncthreads();
        if (broke_down(q)) return false;
    }
    place_diag(NTL - 1);
    __syncthreads();
    return true;
}

// ---------------------------------------------------------------------------
// FP32 tiles

// acc += (NEG ? -1 : 1) * sum_{kk<K} opA[ra+i][ka+kk] * opB[kb+kk][cb+j] with the
// operands rounded to BF16 (round to nearest even) and FP32 accumulation
// (v_mfma_f32_16x16x32_bf16: lane l holds A[l%16][8(l/16)+e] and
// B[8(l/16)+e][l%16], e < 8; accumulator layout as the FP32 tiles).  K is
// padded with zeros to a multiple of 32.
template <int LDA, int LDB, bool TA, bool TB, bool NEG>
__device__ __forceinline__ void mma_tile_bf16(f4& acc, const float* __restrict__ A, int ra, int ka,
                                              const float* __restrict__ B, int cb, int kb, int K) {
    const int lane = threadIdx.x & 63;
    const int i = lane & 15, q = lane >> 4;
    for (int kk = 0; kk < K; kk += 32) {
        bf8 a, b;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = kk + 8 * q + e;
            float av = 0.f, bv = 0.f;
            if (k < K) {
                av = TA ? A[(ka + k) * LDA + ra + i] : A[(ra + i) * LDA + ka + k];
                bv = TB ? B[(cb + i) * LDB + kb + k] : B[(kb + k) * LDB + cb + i];
            }
            a[e] = (__bf16)(NEG ? -av : av);
            b[e] = (__bf16)bv;
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
}

}  // namespace tiles
}  // namespace btc
