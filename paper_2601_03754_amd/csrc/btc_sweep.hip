// Level sweeps of the solve (section "Cholesky Solve", Algorithm 6) on the
// matrix cores: one team of NP/16 wavefronts per node, every n x n block read
// from HBM once, straight into the matrix cores' operand registers.
//
//   forward, node i of level l (stride s), levels ascending:
//     y_i = L_ii^{-1} (b_i - U_{i-s/2} - V_{i+s/2})
//     U_i = R_i y_i + U_{i+s/2}     (everything i's subtree leaves for i+s)
//     V_i = T_i^T y_i + V_{i-s/2}   (everything it leaves for i-s)
//   backward, levels descending:
//     x_i = L_ii^{-T} (y_i - R_i^T x_{i+s} - T_i x_{i-s})
// Instead of two nodes subtracting into the same y concurrently, each node
// takes its two children's sums and passes on theirs with its own (the
// subtree left of a node leaves one vector for it, however many levels it
// has; leaving one per level made a top node gather up to twice its level's
// number of vectors).  Results are deterministic.
//
// A node step of the upper levels is bound by latency, not by traffic: one
// wavefront per node that streams the blocks through LDS slab by slab takes
// 30 to 45 us in FP64 at n = 96 (about 380 cycles for each of its 288 column
// steps: LDS read, lane broadcast, division, update).  Here
//   * all loads of a node (its L, R and T blocks) are in flight at once, in
//     the registers of the team's wavefronts: wavefront w holds tile row w of
//     L and R and tile column w of T (forward; transposed roles backward);
//   * the triangular solve is a chain over 16 x 16 tiles, not over columns:
//     the factor kernels leave the inverse of every diagonal tile in the
//     strict upper part of that tile of L_ii (transposed; its diagonal is
//     1 / L_jj), so a chain step is one product with the inverse and one
//     with the next tile of L, about 300 cycles for 16 columns;
//   * every product runs on the matrix cores (FP64 4x4x4 with four blocks:
//     16 rows by 4 columns in 16 cycles; FP32 16x16x4), which also do the
//     sums over lanes; up to 16 right-hand sides share one pass over the
//     blocks.
//   * the upper levels run in one launch (k_sweep_flow), whose workgroups have
//     their blocks in registers when the vectors they wait for arrive.
// Measured, before and after: N = 4096, n = 96, one right-hand side, FP64:
// forward 560 -> 228 us, backward 480 -> 226 us (level 0, 377 MB: 94 us, 4.0
// TB/s; the nine upper levels in one launch 49 us; a level of 256 nodes 14);
// N = 1023, n = 128, five right-hand sides: whole solve 2 855 -> 291 us.
#include <type_traits>

#include "btc_device.h"
#include "btc_kernels.h"

namespace btc {
namespace {

constexpr unsigned long long kInfoOk = ~0ull;
constexpr int kTl = 16;  // tile side

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// Matrix-core engine of a storage type: a 16 x 16 tile of A times CW columns
// in four instructions.  Lane l holds A[l % 16][k(s)] of step s and B[k(s)][col],
// k(s) = kidx(s, l / 16): the order of k is chosen so that a lane's four
// elements of a row-major tile row are contiguous in pairs (FP64) or all
// four (FP32).  Accumulator register v of lane l: element (row(v), col).
template <class T>
struct Eng;

// v_mfma_f64_4x4x4 with four blocks: block b (lanes 4b .. 4b+3 of every row of
// 16 lanes) multiplies rows 4b .. 4b+3 of the tile with four columns.
template <>
struct Eng<double> {
    static constexpr int CW = 4, NV = 1;
    struct Acc {
        double v[1];
    };
    __device__ static int kidx(int s, int q) { return 8 * (s >> 1) + 2 * q + (s & 1); }
    __device__ static int row(int, int lane) { return (lane & 12) + (lane >> 4); }
    __device__ static int col(int lane) { return lane & 3; }
    __device__ static void mma(Acc& c, double a, double b) {
        c.v[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c.v[0], 0, 0, 0);
    }
    // Product of the diagonal tile's inverse with a vector tile in the
    // accumulator layout: the four blocks of an instruction may take
    // different k ranges, so step s takes in block b the rows 4((b - s) % 4)
    // .. +3, which a rotation of the 16-lane rows by 4s brings there (no LDS
    // round trip).  didx: the k of step s.
    __device__ static int didx(int s, int lane) { return 4 * ((((lane & 15) >> 2) - s) & 3) + (lane >> 4); }
    template <int CTRL>
    __device__ static double rot(double x) {
        const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, false);
        const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, false);
        return __hiloint2double(hi, lo);
    }
    __device__ static Acc dmul(const double (&d)[4], const Acc& x) {
        Acc o;
        o.v[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(d[0], x.v[0], 0.0, 0, 0, 0);
        mma(o, d[1], rot<0x124>(x.v[0]));  // row_ror:4
        mma(o, d[2], rot<0x128>(x.v[0]));  // row_ror:8
        mma(o, d[3], rot<0x12C>(x.v[0]));  // row_ror:12
        return o;
    }
};

template <>
struct Eng<float> {
    static constexpr int CW = 16, NV = 4;
    union Acc {
        f4_t f;
        float v[4];
    };
    __device__ static int kidx(int s, int q) { return 4 * q + s; }
    __device__ static int row(int v, int lane) { return 4 * (lane >> 4) + v; }
    __device__ static int col(int lane) { return lane & 15; }
    __device__ static void mma(Acc& c, float a, float b) {
        c.f = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c.f, 0, 0, 0);
    }
    // the accumulator layout is the B operand layout of k = 4q + s
    __device__ static int didx(int s, int lane) { return 4 * (lane >> 4) + s; }
    __device__ static Acc dmul(const float (&d)[4], const Acc& x) {
        Acc o;
        o.f = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) mma(o, d[s], x.f[s]);
        return o;
    }
};

template <class T>
__device__ __forceinline__ typename Eng<T>::Acc acc_zero() {
    typename Eng<T>::Acc a;
#pragma unroll
    for (int v = 0; v < Eng<T>::NV; ++v) a.v[v] = T(0);
    return a;
}

// All loads of a node go out in straight-line code: a load that does not
// apply (a block the node does not have, a tile past n) gets a scalar offset
// past the resource's end and reads 0 without touching memory.  No branch
// then separates a load from its use, so the compiler's waits count exactly
// the loads that are needed; with branches it waits for every load in flight
// before the first use.

// Loads return in the order they went out: the instruction scheduler is held
// to the order of use.
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0); }

// Lane offsets (bytes) of the tile operands of an n x n block.
template <class T>
struct Lane {
    int rw;     // row-wise: row i of a tile row, first element of the lane's share
    int cw[4];  // column-wise: the lane's elements of column c0 + i, masked past n
    // c0: first column of the column-wise tiles
    __device__ __forceinline__ Lane(int lane, int n, int c0) {
        using E = Eng<T>;
        const int i = lane & 15, q = lane >> 4;
        rw = (i * n + E::kidx(0, q)) * (int)sizeof(T);
#pragma unroll
        for (int s = 0; s < 4; ++s) cw[s] = c0 + i < n ? (E::kidx(s, q) * n + c0 + i) * (int)sizeof(T) : kOob;
    }
};

// Tile operand A[i][k] = M[r0 + i][c0 + k], soff the byte offset of (r0, c0):
// 16-byte loads at element alignment (the blocks are unpadded; range checks
// are per dword).  In the last, partial tile of a row the columns past n are
// elements of the next row: mask_tail.
template <class T>
__device__ __forceinline__ void load_rowwise(T (&a)[4], __amdgpu_buffer_rsrc_t rs, const Lane<T>& ln, int soff) {
    if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x4_t x = __builtin_amdgcn_raw_buffer_load_b128(rs, ln.rw + 64 * h, soff, 0);
            a[2 * h] = __hiloint2double((int)x[1], (int)x[0]);
            a[2 * h + 1] = __hiloint2double((int)x[3], (int)x[2]);
        }
    } else {
        const u32x4_t x = __builtin_amdgcn_raw_buffer_load_b128(rs, ln.rw, soff, 0);
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s] = __int_as_float((int)x[s]);
    }
}
template <class T>
__device__ __forceinline__ void mask_tail(T (&a)[4], int n, int c0, int lane) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (c0 + Eng<T>::kidx(s, lane >> 4) >= n) a[s] = T(0);
}

// Tile operand A[i][k] = M[r0 + k][c0 + i], soff the byte offset of row r0
// (c0 is in ln): lanes read along the rows.
template <class T>
__device__ __forceinline__ void load_colwise(T (&a)[4], __amdgpu_buffer_rsrc_t rs, const Lane<T>& ln, int soff) {
#pragma unroll
    for (int s = 0; s < 4; ++s) buf_ld(a[s], rs, ln.cw[s], soff);
}

// Operand of the inverse of diagonal tile t (TR: its transpose), k order
// didx.  The tile of the stored L_ii holds L in its lower part with the
// diagonal, and the inverse's strict lower part transposed in its strict
// upper part.  The diagonal itself is loaded as L_jj: invert_diag.
template <class T, bool TR>
__device__ __forceinline__ void load_dinv(T (&d)[4], __amdgpu_buffer_rsrc_t rs, int n, int t, int lane) {
    const int i = lane & 15, t0 = kTl * t;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int k = Eng<T>::didx(s, lane);
        // Dinv[i][k], k <= i, at row k, column i; Dinv^T[i][k] = Dinv[k][i],
        // i <= k, at row i, column k
        const int r = t0 + (TR ? i : k), c = t0 + (TR ? k : i);
        buf_ld(d[s], rs, elem_off<T>(r, c, n, r <= c && c < n));
    }
}
template <class T>
__device__ __forceinline__ void invert_diag(T (&d)[4], int n, int t, int lane) {
    const int i = lane & 15;
    T piv = T(1);
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (Eng<T>::didx(s, lane) == i && kTl * t + i < n) piv = d[s];
    const T inv = T(1) / piv;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (Eng<T>::didx(s, lane) == i && kTl * t + i < n) d[s] = inv;
}

// Rows 16w .. 16w+15 of an n x m vector of one node, addressed by byte
// offsets from row 16w; absent: reads 0, writes dropped.
template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t vec_rsrc(const T* v, int n, int m, int64_t node, bool present,
                                                           int w) {
    const int rows = n - kTl * w < kTl ? n - kTl * w : kTl;
    const bool ok = present && rows > 0;
    return block_rsrc(v + (ok ? ((size_t)node * n + kTl * w) * m : 0), ok ? rows * m * (int)sizeof(T) : 0);
}

// Elements of those rows.  At: place of the element in row r, column q (not ok:
// none, reads 0, writes dropped): a byte offset of T's array, or with WIDE, for
// vectors too wide for 32-bit offsets (wide_vectors), an element index.  S may be
// double where T is float.
template <bool WIDE, class T>
struct Rows {
    using At = std::conditional_t<WIDE, int64_t, int>;
    __device__ static At at(bool ok, int r, int m, int q) {
        if constexpr (WIDE) return ok ? (int64_t)r * m + q : -1;
        else return ok ? (r * m + q) * (int)sizeof(T) : kOob;
    }
    template <int AUX = 0, class S>
    __device__ __forceinline__ static void ld(S& x, const S* v, int n, int m, int64_t node, bool present, int w,
                                              At a) {
        if constexpr (WIDE) {
            const S* p = v + ((size_t)node * n + kTl * w) * m + a;
            x = S(0);
            if (present && a >= 0) x = AUX ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
        } else {
            buf_ld<AUX>(x, vec_rsrc(v, n, m, node, present, w), sizeof(S) == sizeof(T) || a == kOob ? a : 2 * a);
        }
    }
    template <int AUX = 0, class S>
    __device__ __forceinline__ static void st(S x, S* v, int n, int m, int64_t node, bool present, int w, At a) {
        if constexpr (WIDE) {
            S* p = v + ((size_t)node * n + kTl * w) * m + a;
            if (!present || a < 0) return;
            if constexpr (AUX) __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *p = x;
        } else {
            buf_st<AUX>(x, vec_rsrc(v, n, m, node, present, w), sizeof(S) == sizeof(T) || a == kOob ? a : 2 * a);
        }
    }
};

template <class T>
__device__ __forceinline__ bool skip_item(const SweepDesc<T>& P) {
    // both flags in one round trip
    typedef const unsigned long long __attribute__((address_space(1)))* gu64;
    typedef const int __attribute__((address_space(1)))* gi32;
    const unsigned long long info = *(gu64)P.info;
    const int skip = *(gi32)(P.skip ? P.skip : (const int*)P.info);
    return info != kInfoOk || (P.skip && skip != 0);
}

// A node's position in the elimination tree.
template <class T>
struct Pos {
    int64_t i, s, pi;
    bool has_r, has_l;
    __device__ __forceinline__ Pos(const SweepDesc<T>& P, int lvl, int64_t kk) {
        s = (int64_t)1 << lvl;
        i = (kk * 2 + 1) << lvl;
        has_r = i + s <= P.N;
        has_l = i > s;
        pi = perm_pos(P.N, lvl, i);
    }
};

// The tree of the sums: node i of level l > 0 takes its left child's (i - s/2)
// and those of the nearest node below on its right, i + 2^l2: the right child,
// or where the chain ends before it the largest 2^l2 still inside.  That
// makes every node the source of exactly one other, its parent.
template <class T>
struct Kin {
    bool left, right;   // children present
    int l2;             // level of the right one
    int64_t pl, pr;     // their positions
    __device__ __forceinline__ Kin(const SweepDesc<T>& P, const Pos<T>& d, int lvl) {
        const int64_t h = d.s >> 1, room = P.N - d.i;
        left = lvl > 0;
        right = lvl > 0 && room > 0;
        l2 = room >= h ? lvl - 1 : room > 0 ? 63 - __builtin_clzll((unsigned long long)room) : 0;
        pl = left ? perm_pos(P.N, lvl - 1, d.i - h) : 0;
        pr = right ? perm_pos(P.N, l2, d.i + ((int64_t)1 << l2)) : 0;
    }
};
// Level of node i's parent (64: none, the root).
template <class T>
__device__ __forceinline__ int parent_level(const Pos<T>& d, int lvl) {
    const int64_t k = d.i >> (lvl + 1);
    if ((k & 1) || d.has_r) return lvl + 1;
    return k == 0 ? 64 : lvl + 1 + __builtin_ctzll((unsigned long long)k);
}

// Several levels in one launch (k_sweep_flow): the nodes of levels l0 .. l1-1,
// one workgroup each, in level order.  A workgroup puts its node's blocks in
// flight, waits for the flags of the nodes it depends on inside the range,
// and sets its own once its vectors are out.  Flags: one word per node and
// direction, set by the producer and cleared by its single reader, so they
// are zero again when a launch ends.
struct Flow {
    int* flag;     // words of this direction, indexed by permuted position
    int l0, l1;
};
constexpr int kCoherent = 16;  // cache policy of vectors exchanged inside a launch: agent scope (sc1)

__device__ __forceinline__ int flag_load(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void flag_store(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The first wavefront waits until flags a and b (null: nothing to wait for)
// are set and clears them; the others wait for it.  The nodes waited for have
// smaller tickets, so they are running or done.  (No bound on the polls: a node
// of millions of right-hand sides works for seconds.)
__device__ __forceinline__ void flow_wait(int* a, int* b, int wave) {
    if (wave == 0 && (a || b)) {
        int* f = (threadIdx.x & 1) ? b : a;
        while (!__all(f == nullptr || flag_load(f) != 0)) __builtin_amdgcn_s_sleep(1);
        if (threadIdx.x < 2 && f) flag_store(f, 0);
    }
    __syncthreads();
}
// Every thread's vector stores (agent scope) have reached memory, then the
// flags are set.
__device__ __forceinline__ void flow_signal(int* a, int* b) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        if (a) flag_store(a, 1);
        if (b) flag_store(b, 1);
    }
}

// Geometry of a team (NP/16 wavefronts, one node) with NG column groups per
// pass.
template <int NP, class T, int NG>
struct Team {
    using E = Eng<T>;
    static constexpr int W = NP / kTl;            // wavefronts = tiles per side
    static constexpr int TH = W * kWave;          // threads
    static constexpr int CP = E::CW * NG;         // columns per pass
    static constexpr int VEC = NP * CP;           // elements of a vector buffer
    static constexpr int LDS(bool bwd) { return bwd ? 3 * VEC : VEC; }  // y, or x and two more vectors
};

// ---------------------------------------------------------------------------
// Forward step of node kk of level lvl by one team (wavefront w of it).
template <int NP, class T, int NG, bool FLOW, bool WIDE>
__device__ __forceinline__ void fwd_team(const SweepDesc<T>& P, int lvl, int64_t kk, int w, T* __restrict__ lds,
                                         const Flow& fl) {
    using G = Team<NP, T, NG>;
    using E = Eng<T>;
    using V = Rows<WIDE, T>;
    constexpr int W = G::W, CP = G::CP, SZ = (int)sizeof(T);
    const int lane = threadIdx.x & (kWave - 1);
    const int n = P.n, m = P.m;
    const size_t nn = (size_t)n * n;
    const Pos<T> d(P, lvl, kk);
    const Kin<T> kin(P, d, lvl);
    const int nt = (n + kTl - 1) / kTl;
    const bool mine = w < nt;  // this wavefront has a tile row
    T* ys = lds;               // y, [row][column of the pass]
    // U of the right child and V of the left child are passed on with the
    // node's own products
    const bool pass_u = lvl > 0 && d.has_r, pass_v = lvl > 0 && d.has_l;

    T Lr[W][4], Rr[W][4], Tr[W][4], Dr[4];
    // one pass over columns q0 .. q0+CP-1; the first one, compiled on its own,
    // loads the blocks (in code shared with the others its waits would have
    // to hold for passes in which no block load follows the vectors)
    auto pass = [&](int q0, auto load) {
        constexpr bool LOAD = decltype(load)::value;
        const int cols = m - q0 < CP ? m - q0 : CP;
        typename E::Acc acc[NG], u[NG], v[NG], sl[NG], sr[NG];
        double b64[NG][E::NV];
        typename V::At vo[NG][E::NV];  // the lane's elements of a node's vectors
        const bool wide = sizeof(T) == 4 && P.B64;  // the right-hand side is FP64
        auto load_rhs = [&]() {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int c = E::CW * g + E::col(lane);
#pragma unroll
                for (int x = 0; x < E::NV; ++x) {
                    const int r = E::row(x, lane);
                    vo[g][x] = V::at(kTl * w + r < n && c < cols, r, m, q0 + c);
                    V::ld(acc[g].v[x], P.B, n, m, d.i - 1, !wide, w, vo[g][x]);
                    if constexpr (SZ == 4) V::ld(b64[g][x], P.B64, n, m, d.i - 1, wide, w, vo[g][x]);
                }
            }
        };
        auto load_sums = [&]() {
            constexpr int AUX = FLOW ? kCoherent : 0;
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int x = 0; x < E::NV; ++x) {
                    V::template ld<AUX>(sl[g].v[x], P.U, n, m, kin.pl, kin.left, w, vo[g][x]);
                    V::template ld<AUX>(sr[g].v[x], P.V, n, m, kin.pr, kin.right, w, vo[g][x]);
                    V::template ld<AUX>(u[g].v[x], P.U, n, m, kin.pr, pass_u, w, vo[g][x]);
                    V::template ld<AUX>(v[g].v[x], P.V, n, m, kin.pl, pass_v, w, vo[g][x]);
                }
        };
        // the vectors go out ahead of the block loads; the children's sums
        // after them where they have to be waited for
        load_rhs();
        if constexpr (!FLOW || !LOAD) load_sums();
        keep_order();
        if constexpr (LOAD) {
            const Lane<T> ln(lane, n, kTl * w);
            const __amdgpu_buffer_rsrc_t lr = block_rsrc(P.Ld + d.pi * nn, mine ? n * n * SZ : 0),
                                         rr = block_rsrc(P.Rb + d.pi * nn, mine && d.has_r ? n * n * SZ : 0),
                                         tr = block_rsrc(P.Tb + d.pi * nn, mine && d.has_l ? n * n * SZ : 0);
            load_dinv<T, false>(Dr, lr, n, w, lane);
            keep_order();
#pragma unroll
            for (int p = 0; p + 1 < W; ++p) load_rowwise(Lr[p], lr, ln, p < w ? (kTl * w * n + kTl * p) * SZ : kOob);
            keep_order();
#pragma unroll
            for (int p = 0; p < W; ++p) {
                load_rowwise(Rr[p], rr, ln, p < nt ? (kTl * w * n + kTl * p) * SZ : kOob);
                load_colwise(Tr[p], tr, ln, p < nt ? kTl * p * n * SZ : kOob);
                keep_order();
            }
            if constexpr (FLOW) {
                flow_wait(kin.left && lvl - 1 >= fl.l0 ? fl.flag + kin.pl : nullptr,
                          kin.right && kin.l2 >= fl.l0 ? fl.flag + kin.pr : nullptr, w);
                load_sums();
            }
        }
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int x = 0; x < E::NV; ++x) {
                if (SZ == 4) acc[g].v[x] += (T)b64[g][x];  // the absent one of the two reads 0
                acc[g].v[x] = (acc[g].v[x] - sl[g].v[x]) - sr[g].v[x];
            }
        if constexpr (LOAD) invert_diag(Dr, n, w, lane);
        // y tile w = Dinv_w acc to LDS for the team
        auto publish = [&]() {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (E::CW * g >= cols) break;
                acc[g] = E::dmul(Dr, acc[g]);
                const int c = E::CW * g + E::col(lane);
#pragma unroll
                for (int x = 0; x < E::NV; ++x) ys[(kTl * w + E::row(x, lane)) * CP + c] = acc[g].v[x];
            }
        };
        if (w == 0) publish();
#pragma unroll
        for (int p = 0; p < W; ++p) {
            if (p >= nt) break;
            __syncthreads();
            if (!mine) continue;
            T b[NG][4];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (E::CW * g >= cols) break;
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    b[g][s] = ys[(kTl * p + E::kidx(s, lane >> 4)) * CP + E::CW * g + E::col(lane)];
            }
            if (p + 1 < W && w > p) {
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    if (E::CW * g >= cols) break;
#pragma unroll
                    for (int s = 0; s < 4; ++s) E::mma(acc[g], Lr[p + 1 < W ? p : 0][s], -b[g][s]);
                }
                // the next tile of the chain before the products off it
                if (w == p + 1) publish();
            }
            if (kTl * p + kTl > n) mask_tail(Rr[p], n, kTl * p, lane);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (E::CW * g >= cols) break;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    E::mma(u[g], Rr[p][s], b[g][s]);
                    E::mma(v[g], Tr[p][s], b[g][s]);
                }
            }
        }
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int x = 0; x < E::NV; ++x) {
                constexpr int AUX = FLOW ? kCoherent : 0;
                V::st(acc[g].v[x], P.Y, n, m, d.pi, true, w, vo[g][x]);
                V::template st<AUX>(u[g].v[x], P.U, n, m, d.pi, d.has_r, w, vo[g][x]);
                V::template st<AUX>(v[g].v[x], P.V, n, m, d.pi, d.has_l, w, vo[g][x]);
            }
    };
    pass(0, std::true_type{});
    for (int q0 = CP; q0 < m; q0 += CP) {
        __syncthreads();  // the vector buffer is free again
        pass(q0, std::false_type{});
    }
    if constexpr (FLOW) flow_signal(parent_level(d, lvl) < fl.l1 ? fl.flag + d.pi : nullptr, nullptr);
}

// ---------------------------------------------------------------------------
// Backward step of node kk of level lvl by one team.
template <int NP, class T, int NG, bool FLOW, bool WIDE>
__device__ __forceinline__ void bwd_team(const SweepDesc<T>& P, int lvl, int64_t kk, int w, T* __restrict__ lds,
                                         const Flow& fl) {
    using G = Team<NP, T, NG>;
    using E = Eng<T>;
    using V = Rows<WIDE, T>;
    constexpr int W = G::W, CP = G::CP, SZ = (int)sizeof(T);
    const int lane = threadIdx.x & (kWave - 1);
    const int n = P.n, m = P.m;
    const size_t nn = (size_t)n * n;
    const Pos<T> d(P, lvl, kk);
    const int nt = (n + kTl - 1) / kTl;
    const bool mine = w < nt;
    T* xs = lds;                 // x, [row][column of the pass]
    T* rs = lds + G::VEC;        // x_{i+s}
    T* ls = lds + 2 * G::VEC;    // x_{i-s}

    T Lr[W][4], Rr[W][4], Tr[W][4], Dr[4];
    auto pass = [&](int q0, auto load) {
        constexpr bool LOAD = decltype(load)::value;
        const int cols = m - q0 < CP ? m - q0 : CP;
        constexpr int PER = kTl * CP / kWave;
        T xr[PER], xl[PER];
        double x0[NG][E::NV];
        typename E::Acc acc[NG];
        typename V::At vo[NG][E::NV];  // the lane's elements of a node's vectors
        // the neighbours' solutions (rows past n: zero)
        auto load_neighbours = [&]() {
            constexpr int AUX = FLOW ? kCoherent : 0;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int e = lane + kWave * k, r = e / CP, c = e % CP;
                const auto at = V::at(kTl * w + r < n && c < cols, r, m, q0 + c);
                V::template ld<AUX>(xr[k], P.X, n, m, d.i + d.s - 1, d.has_r, w, at);
                V::template ld<AUX>(xl[k], P.X, n, m, d.i - d.s - 1, d.has_l, w, at);
            }
        };
        // the vectors go out ahead of the block loads (the neighbours' where
        // they need no wait): the node's y and the iterate it corrects
        if constexpr (!FLOW || !LOAD) load_neighbours();
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int c = E::CW * g + E::col(lane);
#pragma unroll
            for (int x = 0; x < E::NV; ++x) {
                const int r = E::row(x, lane);
                vo[g][x] = V::at(kTl * w + r < n && c < cols, r, m, q0 + c);
                V::ld(acc[g].v[x], P.Y, n, m, d.pi, true, w, vo[g][x]);
                if constexpr (SZ == 4) V::ld(x0[g][x], P.X64, n, m, d.i - 1, P.X64 && !P.first, w, vo[g][x]);
            }
        }
        keep_order();
        if constexpr (LOAD) {
            const Lane<T> ln(lane, n, kTl * w);
            const __amdgpu_buffer_rsrc_t lr = block_rsrc(P.Ld + d.pi * nn, mine ? n * n * SZ : 0),
                                         rr = block_rsrc(P.Rb + d.pi * nn, mine && d.has_r ? n * n * SZ : 0),
                                         tr = block_rsrc(P.Tb + d.pi * nn, mine && d.has_l ? n * n * SZ : 0);
#pragma unroll
            for (int p = 0; p < W; ++p) {
                load_colwise(Rr[p], rr, ln, p < nt ? kTl * p * n * SZ : kOob);
                load_rowwise(Tr[p], tr, ln, p < nt ? (kTl * w * n + kTl * p) * SZ : kOob);
                keep_order();
            }
            load_dinv<T, true>(Dr, lr, n, w, lane);
            keep_order();
#pragma unroll
            for (int p = W - 1; p > 0; --p) {
                load_colwise(Lr[p], lr, ln, p > w && p < nt ? kTl * p * n * SZ : kOob);
                keep_order();
            }
            if constexpr (FLOW) {
                flow_wait(parent_level(d, lvl) < fl.l1 ? fl.flag + d.pi : nullptr, nullptr, w);
                load_neighbours();
            }
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            rs[kTl * CP * w + lane + kWave * k] = xr[k];
            ls[kTl * CP * w + lane + kWave * k] = xl[k];
        }
        __syncthreads();
        auto operand = [&](const T* vec, int p, int g, int s) {
            return vec[(kTl * p + E::kidx(s, lane >> 4)) * CP + E::CW * g + E::col(lane)];
        };
        if (mine) {
#pragma unroll
            for (int p = 0; p < W; ++p) {
                if (p >= nt) break;
                if (kTl * p + kTl > n) mask_tail(Tr[p], n, kTl * p, lane);
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    if (E::CW * g >= cols) break;
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        E::mma(acc[g], Rr[p][s], -operand(rs, p, g, s));
                        E::mma(acc[g], Tr[p][s], -operand(ls, p, g, s));
                    }
                }
            }
        }
        if constexpr (LOAD) invert_diag(Dr, n, w, lane);
        // tile p of x = Dinv_p^T acc to LDS for the team, then its share of the
        // tiles above it
#pragma unroll
        for (int p = W - 1; p >= 0; --p) {
            if (p >= nt) continue;
            if (mine && w == p) {
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    if (E::CW * g >= cols) break;
                    acc[g] = E::dmul(Dr, acc[g]);
                    const int c = E::CW * g + E::col(lane);
#pragma unroll
                    for (int x = 0; x < E::NV; ++x) xs[(kTl * w + E::row(x, lane)) * CP + c] = acc[g].v[x];
                }
            }
            if (p == 0) break;
            __syncthreads();
            if (mine && w < p) {
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    if (E::CW * g >= cols) break;
#pragma unroll
                    for (int s = 0; s < 4; ++s) E::mma(acc[g], Lr[p][s], -operand(xs, p, g, s));
                }
            }
        }
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int x = 0; x < E::NV; ++x) {
                V::template st<FLOW ? kCoherent : 0>(acc[g].v[x], P.X, n, m, d.i - 1, true, w, vo[g][x]);
                if constexpr (SZ == 4)  // (first: the absent iterate reads 0)
                    V::st(x0[g][x] + (double)acc[g].v[x], P.X64, n, m, d.i - 1, P.X64 != nullptr, w, vo[g][x]);
            }
    };
    pass(0, std::true_type{});
    for (int q0 = CP; q0 < m; q0 += CP) {
        __syncthreads();  // the vector buffers are free again
        pass(q0, std::false_type{});
    }
    if constexpr (FLOW) {
        const Kin<T> kin(P, d, lvl);
        flow_signal(kin.left && lvl - 1 >= fl.l0 ? fl.flag + kin.pl : nullptr,
                    kin.right && kin.l2 >= fl.l0 ? fl.flag + kin.pr : nullptr);
    }
}

// ---------------------------------------------------------------------------
// One level of one or many instances: one workgroup (one team) per node.
template <int NP, class T, int NG, bool BWD, bool WIDE>
__global__ __launch_bounds__((Team<NP, T, NG>::TH)) void k_sweep_level(Launch<SweepDesc<T>> L) {
    __shared__ T lds[Team<NP, T, NG>::LDS(BWD)];
    SweepDesc<T> P;
    int lvl;
    int64_t kk;
    fetch_item(L, P, lvl, kk);
    if (skip_item(P)) return;
    const Flow none{nullptr, 0, 0};
    if constexpr (BWD)
        bwd_team<NP, T, NG, false, WIDE>(P, lvl, kk, wave_id(), lds, none);
    else
        fwd_team<NP, T, NG, false, WIDE>(P, lvl, kk, wave_id(), lds, none);
}

// A range of levels in one launch.  The item level field holds l0 | l1 << 8
// and, of explicit items, the node's level << 16; they are in level order
// (forward ascending, backward descending), as are the implicit ones.  The
// workgroups take them by ticket: a workgroup that waits only waits for ones
// that started before it, so the launch always makes progress, whatever the
// dispatch order and whatever else runs on the GPU.  The last ticket resets
// the counter.
template <int NP, class T, int NG, bool BWD, bool WIDE>
__global__ __launch_bounds__((Team<NP, T, NG>::TH)) void k_sweep_flow(Launch<SweepDesc<T>> L) {
    __shared__ T lds[Team<NP, T, NG>::LDS(BWD)];
    __shared__ int slot;
    // a refinement that is done, alone in its launch, skips as a whole, without
    // taking tickets (2048 of them in turn: 25 us instead of 5)
    const bool whole = !L.items && L.single.skip;
    if (whole && skip_item(L.single)) return;
    if constexpr (sizeof(T) == 4)  // (of one instance nothing is looked up: 1 us of 48)
        if (L.items && L.live && *L.live == 0) return;
    if (threadIdx.x == 0) {
        const int t = __hip_atomic_fetch_add(L.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t == (int)gridDim.x - 1) flag_store(L.ticket, 0);
        slot = t;
    }
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(slot);
    if (t < 0 || t >= (int)gridDim.x) return;  // (words shared against the rules)
    SweepDesc<T> P;
    int code, lvl;
    int64_t kk;
    fetch_item_at(L, t, P, code, kk);
    const int l0 = code & 0xff, l1 = (code >> 8) & 0xff;
    if (L.items) {
        lvl = code >> 16;
    } else {
        // position of node t of the range, its level and number
        const int64_t N = P.N, p = BWD ? N - (N >> l1) - 1 - kk : N - (N >> l0) + kk, left = N - p;
        lvl = __builtin_clzll((unsigned long long)left) - __builtin_clzll((unsigned long long)N);
        if ((N >> lvl) < left) --lvl;
        kk = p - (N - (N >> lvl));
    }
    if (!whole && skip_item(P)) return;
    const Flow fl{P.flow, l0, l1};
    if constexpr (BWD)
        bwd_team<NP, T, NG, true, WIDE>(P, lvl, kk, wave_id(), lds, fl);
    else
        fwd_team<NP, T, NG, true, WIDE>(P, lvl, kk, wave_id(), lds, fl);
}

__global__ __launch_bounds__(256) void k_sweep_live(const SweepDesc<float>* __restrict__ descs, int count,
                                                    int* __restrict__ live) {
    bool any = false;
    for (int k = threadIdx.x; k < count; k += 256) any = any || !skip_item(descs[k]);
    const int r = __syncthreads_or(any);
    if (threadIdx.x == 0) *live = r != 0;
}

template <int NP, class T, int NG, bool WIDE = false>
hipError_t launch_ng(const Launch<SweepDesc<T>>& p, int64_t items, bool backward, hipStream_t st, bool flow) {
    const dim3 g((unsigned)items), b(Team<NP, T, NG>::TH);
    if (!flow) {
        if (backward)
            hipLaunchKernelGGL((k_sweep_level<NP, T, NG, true, WIDE>), g, b, 0, st, p);
        else
            hipLaunchKernelGGL((k_sweep_level<NP, T, NG, false, WIDE>), g, b, 0, st, p);
    } else {
        if (backward)
            hipLaunchKernelGGL((k_sweep_flow<NP, T, NG, true, WIDE>), g, b, 0, st, p);
        else
            hipLaunchKernelGGL((k_sweep_flow<NP, T, NG, false, WIDE>), g, b, 0, st, p);
    }
    return hipGetLastError();
}

// Column groups per pass: FP64 one group of four columns, or with more than
// four columns (mc > 4) four of them, two above n = 64 (a node's blocks leave
// registers for no more there); FP32 always one group of 16.
template <int NP>
hipError_t launch_np(const Launch<SweepDesc<double>>& p, int64_t items, bool backward, int mc, hipStream_t st,
                     bool flow) {
    return mc <= 4 ? launch_ng<NP, double, 1>(p, items, backward, st, flow)
                   : launch_ng<NP, double, (NP > 64 ? 2 : 4)>(p, items, backward, st, flow);
}
template <int NP>
hipError_t launch_np(const Launch<SweepDesc<float>>& p, int64_t items, bool backward, int, hipStream_t st,
                     bool flow) {
    return launch_ng<NP, float, 1>(p, items, backward, st, flow);
}

template <class T>
hipError_t launch_sweep_t(const Launch<SweepDesc<T>>& p, int np, int64_t items, bool backward, int mc,
                          hipStream_t st, bool flow, bool wide) {
    // (one instantiation for every n: the padding does not enter the results)
    if (wide) return launch_ng<128, T, 1, true>(p, items, backward, st, flow);
    switch (np) {
        case 8:
        case 16: return launch_np<16>(p, items, backward, mc, st, flow);
        case 32: return launch_np<32>(p, items, backward, mc, st, flow);
        case 48: return launch_np<48>(p, items, backward, mc, st, flow);
        case 64: return launch_np<64>(p, items, backward, mc, st, flow);
        case 80: return launch_np<80>(p, items, backward, mc, st, flow);
        case 96: return launch_np<96>(p, items, backward, mc, st, flow);
        case 128: return launch_np<128>(p, items, backward, mc, st, flow);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_sweep_live(const SweepDesc<float>* descs, int count, int* live, hipStream_t st) {
    hipLaunchKernelGGL(k_sweep_live, dim3(1), dim3(256), 0, st, descs, count, live);
    return hipGetLastError();
}

hipError_t launch_sweep(const Launch<SweepDesc<double>>& p, int np, int64_t items, bool backward, int mc,
                        hipStream_t st, bool flow, bool wide) {
    return launch_sweep_t<double>(p, np, items, backward, mc, st, flow, wide);
}

hipError_t launch_sweep(const Launch<SweepDesc<float>>& p, int np, int64_t items, bool backward, int mc,
                        hipStream_t st, bool flow, bool wide) {
    return launch_sweep_t<float>(p, np, items, backward, mc, st, flow, wide);
}

}  // namespace btc
