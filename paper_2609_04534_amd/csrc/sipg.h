// Device code of the coupled SIPG operator on a uniform Cartesian box mesh
// (shared by sipg.hip, pcg.hip and mg.hip): the face terms, and the row for one
// cell per wave (n >= 5; the row of 64 or 128 cells per workgroup, n <= 4, is in
// tile.h).  One fused kernel computes v = A u with A = A^vol + A^face (Sec. 3, eq. (sipg),
// eq. (operator_split)), homogeneous Dirichlet data imposed by Nitsche's
// terms on the boundary faces.
//
// Row of cell c.  The cell-diagonal block is the Kronecker sum of the cell
// block (eq. (cell_block), A_hat = K_hat + the own-side blocks of both
// interior face stencils) plus, on a boundary face, the difference between
// the Nitsche own-side block and the interior one.  The off-diagonal blocks
// couple c to its face neighbours through N^{-+} and N^{+-} of
// eq. (face_factorized) in the normal slot and the mass matrix in the two
// tangential slots.  With e0, e1 the endpoint values (unit vectors of the
// Gauss-Lobatto basis) and g0, g1 the reference endpoint derivatives, every
// face term is rank two in the normal slot (the rank-two flux structure of
// Sec. 6.3):
//
//   (N w)_i = e_end,i alpha(w) + g_end,i beta(w),    then (x) M (x) M,
//
// where, for the face at the cell's upper end along an axis (normal slot
// index k, source block w):
//   interior:  w = upper neighbour, alpha = -sigma w_0 - 1/2 g0.w,  beta = +1/2 w_0
//   boundary:  w = the cell itself, alpha = -1/2 g1.w,              beta = -1/2 w_{n-1}
// and for the lower end:
//   interior:  w = lower neighbour, alpha = -sigma w_{n-1} + 1/2 g1.w, beta = -1/2 w_{n-1}
//   boundary:  w = the cell itself, alpha = +1/2 g0.w,                 beta = +1/2 w_0
// (sigma = C p (p+1), Sec. 6.2; every term scales with s_d = h_o1 h_o2 / h_d
// like the volume term of that axis).  The face-only operator A^face uses
// A_hat - K_hat for the cell-diagonal Kronecker sum.
//
// Unlike the paper's separate face-exchange sweeps, which read and update
// the output's face layers once per axis, the kernel is cell-centric: every
// cell reads its six neighbours (from cache: the same blocks are its
// neighbours' own inputs) and writes its output block once, so HBM sees one
// read of u and one write of v.  Each interior face is evaluated from both
// sides, which costs arithmetic, not HBM bytes.
//
// Mesh order: cell (cx, cy, cz) is block c = (cx m_y + cy) m_z + cz of the
// blocked layout, so the B cells of a tile are consecutive along z.
#pragma once

#include "eo.h"
#include "mesh.h"
#include "tile.h"

namespace tpfdm {

// DoF index of (normal layer k, tangential a, b) for a face normal to axis D
// (a, b are the two other axes in increasing order).
template <int N, int D>
__device__ __forceinline__ constexpr int fq(int k, int a, int b) {
    return D == 0 ? (k * N + a) * N + b : D == 1 ? (a * N + k) * N + b : (a * N + b) * N + k;
}

// ============================================================ one cell per wave (n >= 5)
// The cell's block lives in an LDS slab (Slab<N> layout, one pencil per lane
// and phase, as in the even-odd wave kernels); the volume product is the
// even-odd LDS apply with the cell-diagonal P_hat, done first.  The six face
// terms are slabs over the two tangential indices, kept in the volume
// product's scratch once that is free: lane (a, b) accumulates alpha and
// beta of every face from the source block's n values along the normal at
// (a, b); the tangential mass M (.) M of all twelve slabs runs as two
// in-place LDS passes of one n-pencil per task (a task owns its row, then
// its column; 12 n tasks per pass spread over the wave); finally lane (j, k)
// adds the face terms to its x-pencil of the volume product.
// The volume product's second scratch slab is the block's own slab s: each
// lane overwrites only the slab positions it has itself just read (its
// pencil in the first phase, its x-pencil in the last), so s, one scratch
// slab and the face slabs are all the LDS a wave needs (10.75 KB at n = 8
// in FP64: 14 waves per CU instead of 11).
template <int N, typename T>
struct WaveLds {
    static constexpr int kT = 12 * N * N > Slab<N>::size ? 12 * N * N : Slab<N>::size;
    T s[Slab<N>::size];          // the cell's block, then its volume product (and scratch t2)
    T t[kT];                     // volume scratch t1, then the twelve face slabs
};

// The lane's x-pencil y[i] = (A u)_c at (i, j, k) with (j, k) = (pc.pa,
// pc.pb), for the active lanes; every lane of the wave must call it.
// TB: ME | MO | PE | PO (even-odd halves of M_hat and of the cell-diagonal
// P_hat); F: endpoint derivatives and the reference penalty.
// HERM: the Hermite-type basis.  The even-odd tables then hold the matrices
// conjugated by D = diag(hermite_sign) (centrosymmetric), so every value is
// multiplied by its sign s(i) s(j) s(k) on load and on store, and the face
// terms read only the layers 0, 1, n-2, n-1 along the normal (the others
// carry no weight: eq. (hermite_traces_3d)).
template <int N, typename T, bool VP, bool HERM = false>
__device__ __forceinline__ void wave_sipg_cell(const T* __restrict__ u, const MeshArgs& G, const T* TB,
                                               const FaceRef<N, T>& F, int64_t c, WaveLds<N, T>& L,
                                               T (&y)[N]) {
    using SL = Slab<N>;
    using S = EOShape<N>;
    constexpr int N3 = N * N * N;
    const T* ME = TB;
    const T* MO = TB + S::SE;
    const T* PE = TB + S::SE + S::SO;
    const T* PO = TB + 2 * S::SE + S::SO;
    const Pencil<N> pc(1);
    const int pa = pc.pa, pb = pc.pb;
    const T* ub = u + G.offset;
    const int lb = G.logB;
    const uint32_t cu = static_cast<uint32_t>(c);
    const uint32_t cz = cu % static_cast<uint32_t>(G.mz);
    const uint32_t rr = cu / static_cast<uint32_t>(G.mz);
    const uint32_t cy = rr % static_cast<uint32_t>(G.my);
    const uint32_t cx = rr / static_cast<uint32_t>(G.my);
    const T sx = static_cast<T>(G.sx), sy = static_cast<T>(G.sy), sz = static_cast<T>(G.sz);
    auto sg = [](int i) { return HERM ? static_cast<T>(hermite_sign(N, i)) : T(1); };
    const T sab = sg(pa) * sg(pb);   // sign of the lane's two tangential indices
    // --- the cell's own block into the slab, volume product in place
    if (pc.act) {
        T x[N];
        pencil_load<N, VP>(x, ub + block_base(c, lb, N3) + (static_cast<int64_t>((pa * N + pb) * N) << lb), lb);
#pragma unroll
        for (int k = 0; k < N; ++k) L.s[SL::at(pa, pb, k)] = HERM ? sab * sg(k) * x[k] : x[k];
    }
    wave_sync();
    eo_apply_lds<N, T>(pc, L.s, L.s, L.t, L.s, ME, MO, PE, PO, sx, sy, sz);   // ends synced
    // --- face slabs in the free scratch: alpha (2 f) and beta (2 f + 1) of
    // face f = 2 axis + upper, slab sl at fs + sl n^2
    T* fs = L.t;
    const int64_t syz = static_cast<int64_t>(G.my) * G.mz;
    auto face = [&](auto Dc, auto UPc, bool interior, int64_t d, T s) {
        constexpr int D = decltype(Dc)::value;
        constexpr bool UP = decltype(UPc)::value;
        constexpr int f = 2 * D + (UP ? 1 : 0);
        const T* w = ub + block_base(interior ? c + d : c, lb, N3);
        const bool first = (UP == interior);
        const T cb0 = first ? T(0.5) * s : T(0);
        const T cbn = first ? T(0) : T(-0.5) * s;
        if (pc.act) {
            // normal to z the n values are the lane's contiguous pencil: one
            // vector load per 16 bytes when VP
            T al = T(0), be = T(0);
            if constexpr (HERM) {
                // two source layers: 0, 1 when the face is interior at the
                // upper end or boundary at the lower end, else n-2, n-1
                // (the weights of the other layers vanish in this basis)
                const int k0 = first ? 0 : N - 2;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int k = k0 + t;
                    T wk = ldc<T>(w + (static_cast<int64_t>(D == 0 ? (k * N + pa) * N + pb
                                                           : D == 1 ? (pa * N + k) * N + pb
                                                                    : (pa * N + pb) * N + k) << lb));
                    wk *= sab * sg(k);
                    // alpha weight of layer k (as below), selected per lane
                    T wgt = T(0);
#pragma unroll
                    for (int kk = 0; kk < N; ++kk) {
                        const T in = UP ? fma(T(-0.5), F.g0[kk], kk == 0 ? -F.sigma : T(0))
                                        : fma(T(0.5), F.g1[kk], kk == N - 1 ? -F.sigma : T(0));
                        const T bd = UP ? T(-0.5) * F.g1[kk] : T(0.5) * F.g0[kk];
                        wgt = kk == k ? s * (interior ? in : bd) : wgt;
                    }
                    al = fma(wgt, wk, al);
                    be = fma(t == 0 ? cb0 : cbn, wk, be);
                }
            } else {
                T wv[N];
                if constexpr (D == 2)
                    pencil_load<N, VP>(wv, w + (static_cast<int64_t>(fq<N, D>(0, pa, pb)) << lb), lb);
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const T in = UP ? fma(T(-0.5), F.g0[k], k == 0 ? -F.sigma : T(0))
                                    : fma(T(0.5), F.g1[k], k == N - 1 ? -F.sigma : T(0));
                    const T bd = UP ? T(-0.5) * F.g1[k] : T(0.5) * F.g0[k];
                    const T wk = D == 2 ? wv[k] : ldc<T>(w + (static_cast<int64_t>(fq<N, D>(k, pa, pb)) << lb));
                    al = fma(s * (interior ? in : bd), wk, al);
                    if (k == 0) be = cb0 * wk;
                    if (k == N - 1) be = fma(cbn, wk, be);
                }
            }
            fs[(2 * f) * N * N + pa * N + pb] = al;
            fs[(2 * f + 1) * N * N + pa * N + pb] = be;
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using BF = std::integral_constant<bool, false>;
    using BT = std::integral_constant<bool, true>;
    face(I0{}, BF{}, cx > 0, -syz, sx);
    face(I0{}, BT{}, cx + 1 < static_cast<uint32_t>(G.mx), syz, sx);
    face(I1{}, BF{}, cy > 0, -static_cast<int64_t>(G.mz), sy);
    face(I1{}, BT{}, cy + 1 < static_cast<uint32_t>(G.my), G.mz, sy);
    face(I2{}, BF{}, cz > 0, -1, sz);
    face(I2{}, BT{}, cz + 1 < static_cast<uint32_t>(G.mz), 1, sz);
    wave_sync();
    // --- tangential mass of the twelve slabs: rows (second index), then columns
    constexpr int HC = S::HC, H = S::H;
    auto mass_pencil = [&](const T (&xin)[N], T (&out)[N]) {
        T e[HC], o[H], E[HC], O[H];
        eo_split<N>(xin, e, o);
        eo_mul<N>(ME, MO, e, o, E, O);
        eo_join<N>(E, O, out);
    };
    for (int task = threadIdx.x; task < 12 * N; task += 64) {
        const int sl = task / N, a = task - (task / N) * N;
        T xin[N], out[N];
#pragma unroll
        for (int b = 0; b < N; ++b) xin[b] = fs[sl * N * N + a * N + b];
        mass_pencil(xin, out);
#pragma unroll
        for (int b = 0; b < N; ++b) fs[sl * N * N + a * N + b] = out[b];
    }
    wave_sync();
    for (int task = threadIdx.x; task < 12 * N; task += 64) {
        const int sl = task / N, b = task - (task / N) * N;
        T xin[N], out[N];
#pragma unroll
        for (int a = 0; a < N; ++a) xin[a] = fs[sl * N * N + a * N + b];
        mass_pencil(xin, out);
#pragma unroll
        for (int a = 0; a < N; ++a) fs[sl * N * N + a * N + b] = out[a];
    }
    wave_sync();
    // --- the lane's x-pencil of the volume product plus the face terms
    if (pc.act) {
        const int j = pa, k = pb;
        T g0j = T(0), g1j = T(0), g0k = T(0), g1k = T(0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            g0j = j == i ? F.g0[i] : g0j;
            g1j = j == i ? F.g1[i] : g1j;
            g0k = k == i ? F.g0[i] : g0k;
            g1k = k == i ? F.g1[i] : g1k;
        }
        const T ej0 = j == 0 ? T(1) : T(0), ejn = j == N - 1 ? T(1) : T(0);
        const T ek0 = k == 0 ? T(1) : T(0), ekn = k == N - 1 ? T(1) : T(0);
        const T ax0 = fs[0 * N * N + j * N + k], bx0 = fs[1 * N * N + j * N + k];
        const T ax1 = fs[2 * N * N + j * N + k], bx1 = fs[3 * N * N + j * N + k];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            T v = L.s[SL::at(i, j, k)];
            v = fma(F.g0[i], bx0, fma(F.g1[i], bx1, v));                       // x faces, beta
            if (i == 0) v += ax0;                                               // x faces, alpha
            if (i == N - 1) v += ax1;
            v = fma(ej0, fs[4 * N * N + i * N + k], v);                             // y faces
            v = fma(g0j, fs[5 * N * N + i * N + k], v);
            v = fma(ejn, fs[6 * N * N + i * N + k], v);
            v = fma(g1j, fs[7 * N * N + i * N + k], v);
            v = fma(ek0, fs[8 * N * N + i * N + j], v);                             // z faces
            v = fma(g0k, fs[9 * N * N + i * N + j], v);
            v = fma(ekn, fs[10 * N * N + i * N + j], v);
            v = fma(g1k, fs[11 * N * N + i * N + j], v);
            y[i] = HERM ? sab * sg(i) * v : v;
        }
    }
    wave_sync();
}

}  // namespace tpfdm
