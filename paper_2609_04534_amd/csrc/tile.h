// Row of the coupled SIPG operator for consecutive cells of a mesh plan by
// one workgroup of N waves (n <= 4): lane l of every wave holds W consecutive
// cells (64 W cells per workgroup) and wave w an N x N plane of each cell's
// N^3 values.
//
// The row of eq. (sipg) is a sum of three Kronecker terms, one per axis, in
// which that axis' slot holds a 1D operator B_d reaching into the two face
// neighbours and the two other slots hold the mass.  B_d acts on one pencil
// (and the neighbour's pencil behind it), so it is applied to the raw values
// first and every tangential mass runs once on the sum:
//   v = (I (x) M (x) M) B_x u + (M (x) I (x) I) [ (I (x) I (x) M) B_y u + (I (x) M (x) I) B_z u ]
// (B_d scaled by s_d): eight 1D contractions per block and no separate mass
// passes for the face terms.
//
// Roles: wave w works on the x-z plane j = w for the x contractions and on
// the y-z plane i = w for the y and z ones; the planes change hands through
// one LDS block of N^3 x 64 W values (element [q][cell]: every access is
// consecutive words).
//
// What is read from memory: the own block once, the x and y neighbours'
// blocks once each; z neighbours are the adjacent lanes, so their face
// values come by lane shifts, and only the first and last lane of a wave
// load a neighbour's rows.  The kernels are bound by the vector cache: loads
// of 8 bytes a lane run at half its rate (70 bytes per ns and CU against 134
// with 16 bytes, measured on blocks resident in L2), so in FP64 a lane takes
// two cells (W = 2, 16-byte loads) where cell pairs stay together.
#pragma once

#include <type_traits>

#include "mesh.h"

namespace tpfdm {

using ::fma;

// Barrier of a tile workgroup around an LDS exchange: orders LDS only, so
// global loads and stores stay in flight across it.
__device__ __forceinline__ void tile_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One value of each of a lane's W cells.
template <typename T, int W>
struct Cells {
    T v[W];
};
template <typename T, int W>
__device__ __forceinline__ Cells<T, W> zero_cells() {
    Cells<T, W> r;
#pragma unroll
    for (int e = 0; e < W; ++e) r.v[e] = T(0);
    return r;
}
// r = a b + c with a shared by the cells
template <typename T, int W>
__device__ __forceinline__ Cells<T, W> fma(T a, const Cells<T, W>& b, const Cells<T, W>& c) {
    Cells<T, W> r;
#pragma unroll
    for (int e = 0; e < W; ++e) r.v[e] = ::fma(a, b.v[e], c.v[e]);
    return r;
}
template <typename T, int W>
__device__ __forceinline__ Cells<T, W> operator*(T a, const Cells<T, W>& b) {
    Cells<T, W> r;
#pragma unroll
    for (int e = 0; e < W; ++e) r.v[e] = a * b.v[e];
    return r;
}
template <typename T, int W>
__device__ __forceinline__ Cells<T, W> operator+(const Cells<T, W>& a, const Cells<T, W>& b) {
    Cells<T, W> r;
#pragma unroll
    for (int e = 0; e < W; ++e) r.v[e] = a.v[e] + b.v[e];
    return r;
}
template <typename T, int W>
__device__ __forceinline__ Cells<T, W> neg(const Cells<T, W>& a) {
    Cells<T, W> r;
#pragma unroll
    for (int e = 0; e < W; ++e) r.v[e] = -a.v[e];
    return r;
}
// Forces the values to be computed here: the compiler would otherwise sink
// arithmetic below later loads (past scheduling barriers) and keep all that
// was loaded live at once.
template <typename T, int W, int K>
__device__ __forceinline__ void pin(Cells<T, W> (&a)[K]) {
#pragma unroll
    for (int q = 0; q < K; ++q)
#pragma unroll
        for (int e = 0; e < W; ++e) asm volatile("" : "+v"(a[q].v[e]));
}
// The lane's W consecutive values at p (one 2 sizeof(T)-byte access for W = 2).
template <typename TC, int W, typename TS>
__device__ __forceinline__ Cells<TC, W> ld_cells(const TS* p) {
    Cells<TC, W> r;
    if constexpr (W == 1) {
        r.v[0] = ldc<TC>(p);
    } else {
        typedef TS Vec __attribute__((ext_vector_type(W)));
        const Vec t = *reinterpret_cast<const Vec*>(p);
#pragma unroll
        for (int e = 0; e < W; ++e) r.v[e] = static_cast<TC>(t[e]);
    }
    return r;
}
template <bool NT, typename TS, typename TC, int W>
__device__ __forceinline__ void st_cells(TS* p, const Cells<TC, W>& a) {
    if constexpr (W == 1) {
        stv<NT>(p, a.v[0]);
    } else {
        typedef TS Vec __attribute__((ext_vector_type(W)));
        Vec t;
#pragma unroll
        for (int e = 0; e < W; ++e) t[e] = static_cast<TS>(a.v[e]);
        if constexpr (NT) __builtin_nontemporal_store(t, reinterpret_cast<Vec*>(p));
        else *reinterpret_cast<Vec*>(p) = t;
    }
}

// A lane's cells: c .. c + W - 1, and their place in the mesh (W = 2: the
// cells of a pair differ in z only, which needs an even cell count in z).
// Lanes past the last cell compute on the last cells (in bounds) and store
// nothing.  w: the wave's plane index.
template <int W>
struct TileCell {
    int lane, w;
    bool valid;
    int64_t c;
    uint32_t cx, cy, cz;
    __device__ __forceinline__ TileCell(const MeshArgs& G, unsigned tile) {
        lane = threadIdx.x;
        w = __builtin_amdgcn_readfirstlane(threadIdx.y);
        const int64_t g = (static_cast<int64_t>(tile) * 64 + lane) * W;
        valid = g < G.ncells;
        c = valid ? g : G.ncells - W;
        const uint32_t cu = static_cast<uint32_t>(c);
        cz = cu % static_cast<uint32_t>(G.mz);
        const uint32_t rr = cu / static_cast<uint32_t>(G.mz);
        cy = rr % static_cast<uint32_t>(G.my);
        cx = rr / static_cast<uint32_t>(G.my);
    }
};

// Entry (i, j) of a 1D table read through its symmetry class (symmetric, and
// in the Lagrange basis centrosymmetric), so the compiler holds one scalar
// register pair per distinct value.
template <int N, bool HERM>
__host__ __device__ constexpr int sym_index(int i, int j) {
    int a = i < j ? i : j, b = i < j ? j : i;
    if (!HERM && a + b > N - 1) {
        const int t = N - 1 - b;
        b = N - 1 - a;
        a = t;
    }
    return a * N + b;
}

// 1D tables of a tile row: mass M and cell-diagonal operator P, half the
// endpoint derivatives h0 = g0 / 2 (h1 = -h0 reversed in the Lagrange basis;
// in the Hermite-type basis each has one nonzero entry, h0[1] and h1[n-2]),
// and the penalty sigma.
template <int N, typename TC, bool HERM>
struct TileTab {
    TC m[N * N], p[N * N], h0[N], h1[N], sigma;
    __device__ __forceinline__ TC M(int i, int j) const { return m[sym_index<N, HERM>(i, j)]; }
    __device__ __forceinline__ TC P(int i, int j) const { return p[sym_index<N, HERM>(i, j)]; }
    __device__ __forceinline__ TC half_g(bool up, int k) const {
        if (HERM) return up ? h1[k] : h0[k];
        return up ? -h0[N - 1 - k] : h0[k];
    }
    // whether layer k carries a weight of the endpoint derivative
    static constexpr bool has_g(bool up, int k) { return !HERM || k == (up ? N - 2 : 1); }
    // sum_k half_g(up, k) x_k
    template <int W>
    __device__ __forceinline__ Cells<TC, W> half_d(bool up, const Cells<TC, W>* x) const {
        constexpr int k0 = HERM ? 1 : 0;
        if (HERM) return half_g(up, up ? N - 2 : k0) * x[up ? N - 2 : k0];
        Cells<TC, W> d = half_g(up, 0) * x[0];
#pragma unroll
        for (int k = 1; k < N; ++k) d = fma(half_g(up, k), x[k], d);
        return d;
    }
};

// A face adds e_end,k alpha + g_end,k beta to layer k of the cell's pencil
// (see sipg.h).  With the factor 1/2 moved to the derivatives and t the
// trace of the neighbour's pencil w at the face:
//   lower face:  alpha = h1.w - sigma t,   beta' = -t (t = w_{n-1});  boundary: alpha = h0.x,  beta' = x_0
//   upper face:  alpha = -h0.w - sigma t,  beta' = t (t = w_0);       boundary: alpha = -h1.x, beta' = -x_{n-1}
// (x: the cell's own pencil) and layer k gets e_end,k alpha + half_g(up, k) beta'.
// y_k = s (P x + both faces)_k for one pencil of a lane's cells.
template <int N, typename TC, int W, bool HERM>
__device__ __forceinline__ void pencil_row(const TileTab<N, TC, HERM>& R, const Cells<TC, W>* x,
                                           const Cells<TC, W>& al, const Cells<TC, W>& bl, const Cells<TC, W>& ah,
                                           const Cells<TC, W>& bh, TC s, Cells<TC, W> (&y)[N]) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
        Cells<TC, W> v = R.P(r, 0) * x[0];
#pragma unroll
        for (int k = 1; k < N; ++k) v = fma(R.P(r, k), x[k], v);
        if (r == 0) v = v + al;
        if (r == N - 1) v = v + ah;
        if (R.has_g(false, r)) v = fma(R.half_g(false, r), bl, v);
        if (R.has_g(true, r)) v = fma(R.half_g(true, r), bh, v);
        y[r] = s * v;
    }
}

// The value of the previous (UP: next) lane; the first (last) lane of the
// wave gets edge.
template <bool UP>
__device__ __forceinline__ int lane_shift(int v, int edge) {
    return __builtin_amdgcn_update_dpp(edge, v, UP ? 0x130 : 0x138, 0xf, 0xf, false);
}
template <bool UP>
__device__ __forceinline__ float lane_shift(float v, float edge) {
    return __int_as_float(lane_shift<UP>(__float_as_int(v), __float_as_int(edge)));
}
template <bool UP>
__device__ __forceinline__ double lane_shift(double v, double edge) {
    return __hiloint2double(lane_shift<UP>(__double2hiint(v), __double2hiint(edge)),
                            lane_shift<UP>(__double2loint(v), __double2loint(edge)));
}

// The x or y face neighbours of a lane's cells, one pencil (plane index k) at
// a time: the neighbours' source layers of pencil k + 1 are in flight while
// pencil k is worked on (left alone the compiler issues the loads of all
// pencils at once and spills).  ST: stride of the normal index.
template <int N, int ST, typename TS, typename TC, int W, int LB, bool HERM>
struct FaceStream {
    using V = Cells<TC, W>;
    static constexpr int L = HERM ? 2 : N;       // source layers of a face
    static constexpr int kLo = N - L;            // first source layer of the lower neighbour
    const TS *pl, *ph;
    bool lo, hi, inner;
    int lb;
    V nl[2][L], nh[2][L];
    __device__ __forceinline__ FaceStream(const TS* own, bool lo_, bool hi_, int64_t dl, int64_t dh, int lb_)
        : pl(own + (lo_ ? dl : 0)), ph(own + (hi_ ? dh : 0)), lo(lo_), hi(hi_), inner(__all(lo_ && hi_)), lb(lb_) {}
    __device__ __forceinline__ void fetch(int k) {
        const int l = LB >= 0 ? LB : lb;
#pragma unroll
        for (int t = 0; t < L; ++t)
            nl[k & 1][t] = ld_cells<TC, W>(pl + (static_cast<int64_t>((kLo + t) * ST + k) << l));
#pragma unroll
        for (int t = 0; t < L; ++t) nh[k & 1][t] = ld_cells<TC, W>(ph + (static_cast<int64_t>(t * ST + k) << l));
    }
    // y = s (P x + faces) for pencil k; x: the cells' own pencil
    __device__ __forceinline__ void row(const TileTab<N, TC, HERM>& R, int k, const V (&x)[N], TC s, V (&y)[N]) {
        if (k + 1 < N) fetch(k + 1);
        __builtin_amdgcn_sched_barrier(0);
        const V* wl = nl[k & 1];   // layers kLo .. N - 1 of the lower neighbour
        const V* wh = nh[k & 1];   // layers 0 .. L - 1 of the upper one
        V al = -R.sigma * wl[L - 1], ah = -R.sigma * wh[0];
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (R.has_g(true, kLo + t)) al = fma(R.half_g(true, kLo + t), wl[t], al);
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (R.has_g(false, t)) ah = fma(-R.half_g(false, t), wh[t], ah);
        V bl = neg(wl[L - 1]), bh = wh[0];
        if (!inner) {   // some lane's face lies on the boundary
            const V d0 = R.half_d(false, x), d1 = R.half_d(true, x);
#pragma unroll
            for (int e = 0; e < W; ++e) {
                al.v[e] = lo ? al.v[e] : d0.v[e];
                bl.v[e] = lo ? bl.v[e] : x[0].v[e];
                ah.v[e] = hi ? ah.v[e] : -d1.v[e];
                bh.v[e] = hi ? bh.v[e] : -x[N - 1].v[e];
            }
        }
        pencil_row<N, TC, W, HERM>(R, x, al, bl, ah, bh, s, y);
    }
};

// The wave's plane i = w of (A u) for the lane's cells into out (out[j N + k]);
// every thread of the workgroup calls it.  A: N^3 x 64 W values of LDS; on
// return the wave's own plane i = w of A is free for it, the rest after the
// next tile_sync.
template <int N, typename TS, typename TC, int W, int LB, bool HERM>
__device__ __forceinline__ void tile_sipg(const TS* __restrict__ u, const MeshArgs& G,
                                          const TileTab<N, TC, HERM>& R, const TileCell<W>& T,
                                          Cells<TC, W> (*A)[64], Cells<TC, W> (&out)[N * N]) {
    using V = Cells<TC, W>;
    constexpr int N2 = N * N, N3 = N * N * N;
    const int lb = LB >= 0 ? LB : G.logB;
    const int w = T.w, lane = T.lane;
    const int64_t syz = static_cast<int64_t>(G.my) * G.mz;
    const int64_t base = block_base(T.c, lb, N3);
    const TS* ub = u + G.offset + base;
    auto delta = [&](int64_t d) { return block_base(T.c + d, lb, N3) - base; };
    // --- the own y-z plane i = w, kept and shared through LDS
    V own[N2];
    {
        const TS* p = ub + (static_cast<int64_t>(w * N2) << lb);
#pragma unroll
        for (int q = 0; q < N2; ++q) own[q] = ld_cells<TC, W>(p + (static_cast<int64_t>(q) << lb));
    }
    // z neighbours of the first and last lane's cells (in other waves' lanes):
    // alpha and trace of their rows
    TC ea[N], et[N];
#pragma unroll
    for (int j = 0; j < N; ++j) ea[j] = et[j] = TC(0);
    {
        const bool e0 = lane == 0 && T.cz > 0;
        const bool e1 = lane == 63 && T.cz + W < static_cast<uint32_t>(G.mz);
        if (e0 || e1) {
            const TS* p = u + G.offset + block_base(e0 ? T.c - 1 : T.c + W, lb, N3) + (static_cast<int64_t>(w * N2) << lb);
            auto ld = [&](int q) { return ldc<TC>(p + (static_cast<int64_t>(q) << lb)); };
#pragma unroll
            for (int j = 0; j < N; ++j) {
                TC d;
                if constexpr (HERM) {
                    d = (e0 ? R.half_g(true, N - 2) : R.half_g(false, 1)) * ld(j * N + (e0 ? N - 2 : 1));
                    et[j] = ld(j * N + (e0 ? N - 1 : 0));
                } else {
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        const TC cf = e0 ? R.half_g(true, k) : R.half_g(false, k);
                        const TC v = ld(j * N + k);
                        d = k == 0 ? cf * v : fma(cf, v, d);
                        if (k == 0) et[j] = v;
                        if (k == N - 1) et[j] = e0 ? v : et[j];
                    }
                }
                ea[j] = e0 ? fma(-R.sigma, et[j], d) : -fma(R.sigma, et[j], d);
            }
        }
    }
    FaceStream<N, N, TS, TC, W, LB, HERM> fy(ub + (static_cast<int64_t>(w * N2) << lb), T.cy > 0,
                                             T.cy + 1 < static_cast<uint32_t>(G.my), delta(-int64_t(G.mz)),
                                             delta(G.mz), lb);
    fy.fetch(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < N2; ++q) A[w * N2 + q][lane] = own[q];
    // --- y-z plane i = w: ws = M_y B_z u + M_z B_y u
    V ws[N2];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const V* x = own + j * N;
        const V d0 = R.half_d(false, x), d1 = R.half_d(true, x);
        // alphas this cell sends to its upper (au) and lower (ad) neighbour
        const V au = fma(-R.sigma, x[N - 1], d1);
        const V ad = neg(fma(R.sigma, x[0], d0));
        V al, bl, ah, bh;
#pragma unroll
        for (int e = 0; e < W; ++e) {
            const TC pa = e == 0 ? lane_shift<false>(au.v[W - 1], ea[j]) : au.v[e == 0 ? 0 : e - 1];
            const TC pt = e == 0 ? lane_shift<false>(x[N - 1].v[W - 1], et[j]) : x[N - 1].v[e == 0 ? 0 : e - 1];
            const TC na = e == W - 1 ? lane_shift<true>(ad.v[0], ea[j]) : ad.v[e == W - 1 ? 0 : e + 1];
            const TC nt = e == W - 1 ? lane_shift<true>(x[0].v[0], et[j]) : x[0].v[e == W - 1 ? 0 : e + 1];
            const bool lo = T.cz + e > 0, hi = T.cz + e + 1 < static_cast<uint32_t>(G.mz);
            al.v[e] = lo ? pa : d0.v[e];
            bl.v[e] = lo ? -pt : x[0].v[e];
            ah.v[e] = hi ? na : -d1.v[e];
            bh.v[e] = hi ? nt : -x[N - 1].v[e];
        }
        V y[N];
        pencil_row<N, TC, W, HERM>(R, x, al, bl, ah, bh, static_cast<TC>(G.sz), y);
#pragma unroll
        for (int jj = 0; jj < N; ++jj)
#pragma unroll
            for (int k = 0; k < N; ++k)
                ws[jj * N + k] = j == 0 ? R.M(jj, 0) * y[k] : fma(R.M(jj, j), y[k], ws[jj * N + k]);
        pin(ws);
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        V x[N], y[N];
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = own[j * N + k];
        fy.row(R, k, x, static_cast<TC>(G.sy), y);
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int kk = 0; kk < N; ++kk) ws[j * N + kk] = fma(R.M(kk, k), y[j], ws[j * N + kk]);
        pin(ws);
    }
    // --- x-z plane j = w: M_z B_x u, in place
    {
        FaceStream<N, N2, TS, TC, W, LB, HERM> fx(ub + (static_cast<int64_t>(w * N) << lb), T.cx > 0,
                                                  T.cx + 1 < static_cast<uint32_t>(G.mx), delta(-syz), delta(syz), lb);
        fx.fetch(0);
        __builtin_amdgcn_sched_barrier(0);
        tile_sync();
        V tx[N2];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            V x[N], y[N];
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = A[(i * N + w) * N + k][lane];
            fx.row(R, k, x, static_cast<TC>(G.sx), y);
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int kk = 0; kk < N; ++kk)
                    tx[i * N + kk] = k == 0 ? R.M(kk, 0) * y[i] : fma(R.M(kk, k), y[i], tx[i * N + kk]);
            pin(tx);
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k < N; ++k) A[(i * N + w) * N + k][lane] = tx[i * N + k];
    }
    tile_sync();
    // --- plane i = w: out = M_y of the x term; ws takes its place in LDS
    {
        V x[N2];
#pragma unroll
        for (int q = 0; q < N2; ++q) x[q] = A[w * N2 + q][lane];
#pragma unroll
        for (int q = 0; q < N2; ++q) A[w * N2 + q][lane] = ws[q];
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int k = 0; k < N; ++k) {
                V s = R.M(j, 0) * x[k];
#pragma unroll
                for (int jj = 1; jj < N; ++jj) s = fma(R.M(j, jj), x[jj * N + k], s);
                out[j * N + k] = s;
            }
    }
    tile_sync();
    // --- x-z plane j = w: M along x, in place
    {
        V x[N2];
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k < N; ++k) x[i * N + k] = A[(i * N + w) * N + k][lane];
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k < N; ++k) {
                V s = R.M(i, 0) * x[k];
#pragma unroll
                for (int ii = 1; ii < N; ++ii) s = fma(R.M(i, ii), x[ii * N + k], s);
                A[(i * N + w) * N + k][lane] = s;
            }
    }
    tile_sync();
#pragma unroll
    for (int q = 0; q < N2; ++q) out[q] = out[q] + A[w * N2 + q][lane];
}

// Waves per SIMD the tile kernels are built for.  n = 4 in FP64 with one
// cell a lane needs 140 registers (four waves spill: 72 against 94 us on 64^3
// cells); two cells a lane take up to all 256 of two waves (the Lagrange
// kernels of n = 4 spill four to seven values).
template <int N, typename TC, int W>
constexpr int tile_waves() {
    return W == 2 ? 2 : (N == 4 && sizeof(TC) == 8 ? 3 : 4);
}

// Sum of a double over the workgroup (fixed order), for thread (0, 0).
template <int N>
__device__ __forceinline__ double tile_sum(double v, double* red) {
    v = wave_sum(v);
    if (threadIdx.x == 0) red[threadIdx.y] = v;
    tile_sync();
    double s = red[0];
#pragma unroll
    for (int i = 1; i < N; ++i) s += red[i];
    return s;
}

// 1D transform tables of the block inverse: S, and the n^3
// reciprocals 1 / (lam_i s_x + lam_j s_y + lam_k s_z), the same for every
// cell of a uniform mesh.
template <int N, typename TI>
struct TileInv {
    TI s[N * N];
    TI d[N * N * N];
};

// v <- D^{-1} v for the lane's cells, v the plane i = w in
// and out (fast diagonalization: S^T along z and y in the plane, along x
// through LDS, the scaling, and back).  A: N^3 x 64 W values of TI, whose
// plane i = w the wave owns on entry (and again on return).
template <int N, typename TI, int W>
__device__ __forceinline__ void tile_fdm(const TileInv<N, TI>& E, const TileCell<W>& T, Cells<TI, W> (*A)[64],
                                         Cells<TI, W> (&v)[N * N]) {
    using V = Cells<TI, W>;
    constexpr int N2 = N * N;
    const int w = T.w, lane = T.lane;
    // v_c <- sum_k S[k][c] v_k (fwd) or v_k <- sum_c S[k][c] v_c along a pencil
    auto pencil = [&](V(&x)[N2], int base, int st, bool fwd) {
        V t[N];
#pragma unroll
        for (int c = 0; c < N; ++c) {
            V a = (fwd ? E.s[c] : E.s[c * N]) * x[base];
#pragma unroll
            for (int k = 1; k < N; ++k) a = fma(fwd ? E.s[k * N + c] : E.s[c * N + k], x[base + k * st], a);
            t[c] = a;
        }
#pragma unroll
        for (int c = 0; c < N; ++c) x[base + c * st] = t[c];
    };
#pragma unroll
    for (int j = 0; j < N; ++j) pencil(v, j * N, 1, true);
#pragma unroll
    for (int k = 0; k < N; ++k) pencil(v, k, N, true);
#pragma unroll
    for (int q = 0; q < N2; ++q) A[w * N2 + q][lane] = v[q];
    tile_sync();
    {
        V x[N2];   // x-z plane j = w: x[i * N + k]
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k < N; ++k) x[i * N + k] = A[(i * N + w) * N + k][lane];
#pragma unroll
        for (int k = 0; k < N; ++k) pencil(x, k, N, true);
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k < N; ++k) x[i * N + k] = E.d[(i * N + w) * N + k] * x[i * N + k];
#pragma unroll
        for (int k = 0; k < N; ++k) pencil(x, k, N, false);
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k < N; ++k) A[(i * N + w) * N + k][lane] = x[i * N + k];
    }
    tile_sync();
#pragma unroll
    for (int q = 0; q < N2; ++q) v[q] = A[w * N2 + q][lane];
#pragma unroll
    for (int k = 0; k < N; ++k) pencil(v, k, N, false);
#pragma unroll
    for (int j = 0; j < N; ++j) pencil(v, j * N, 1, false);
}

// The tables of a tile row from the plan's reference data.
template <int N, typename TC, bool HERM>
TileTab<N, TC, HERM> tile_tab(const Plan& plan, bool face_only) {
    Pair<N, double> P;
    FaceRef<N, double> F;
    sipg_tables<N, double>(plan, face_only, P, F);
    TileTab<N, TC, HERM> R;
    for (int e = 0; e < N * N; ++e) R.m[e] = static_cast<TC>(P.m[e]), R.p[e] = static_cast<TC>(P.p[e]);
    for (int k = 0; k < N; ++k) R.h0[k] = static_cast<TC>(0.5 * F.g0[k]), R.h1[k] = static_cast<TC>(0.5 * F.g1[k]);
    R.sigma = static_cast<TC>(F.sigma);
    return R;
}

// Whether a lane takes two cells (16-byte loads): FP64, pairs that stay
// together (B = 64, an even cell count in z, 16-byte aligned vectors), and
// enough cells that workgroups of 128 still cover the CUs.  Operator in FP64,
// one against two cells a lane: 128^3 cells n = 2 76 / 48 us, n = 3 293 / 244
// us, n = 4 713 / 550 us; 100^3 n = 4 338 / 300 us; 64^3 n = 2 9.8 / 8.6 us, n =
// 4 68 / 72 us; 32^3 n = 3 8.4 / 8.7 us, n = 4 10.9 / 11.4 us; with an earlier
// form of the row 8^3 cells n = 4 9.1 / 12.0 us.  FP32 loads (4 bytes a lane)
// already run at the full rate and keep one cell.
inline bool tile_pairs(const MeshArgs& G, size_t elem, bool aligned) {
    constexpr int64_t kMinCells = 32768;
    return elem == 8 && aligned && G.logB == 6 && G.offset % 2 == 0 && G.mz % 2 == 0 && G.ncells >= kMinCells;
}
// Workgroups of a tile kernel over a mesh's cells.
inline unsigned tile_grid(const MeshArgs& G, int W) { return static_cast<unsigned>((G.ncells + 64 * W - 1) / (64 * W)); }

// Tables of D^{-1} on a mesh level with the scalings of G, formed in
// FP64 and rounded once.
template <int N, typename TI>
TileInv<N, TI> tile_inv(const RefData& ref, const MeshArgs& G) {
    TileInv<N, TI> E;
    for (int e = 0; e < N * N; ++e) E.s[e] = static_cast<TI>(ref.S[e]);
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j)
            for (int k = 0; k < N; ++k)
                E.d[(i * N + j) * N + k] =
                    static_cast<TI>(1.0 / (ref.lam[i] * G.sx + ref.lam[j] * G.sy + ref.lam[k] * G.sz));
    return E;
}

}  // namespace tpfdm
