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

// ============================================================ one cell per wave (n >= 5)
// The cell's block moves through LDS slabs (Slab<N> layout, one pencil per
// lane and phase, as in the even-odd wave kernels).  With B_d the 1D operator
// of axis d including its two faces, the row is
//   v = B_x a' + M_x b,  a' = M_y M_z u,  b = s_y B_y (M_z u) + s_z M_y (B_z u),
// where the face part of B_z acts on the lane's own z-pencils (and the
// neighbours' behind them) before any mass, and the face parts of B_y and
// B_x, which need the neighbours' values under M_z (and M_y), are carried as
// four slabs per axis over the two tangential indices: lane (a, b) forms them
// from the neighbours' n values along the normal, M_z runs on all eight slabs
// in one pass (8 n row tasks), M_y on the four x slabs, and each lane then
// adds its four values in the even and odd halves of its y- or x-pencil.
// (Twelve slabs through both masses and added to the finished row took 28
// LDS passes of a block against 13 here; the kernel was bound by LDS, 83% of
// its time at n = 8 in FP64.)
template <int N, typename T>
struct WaveLds {
    static constexpr int kFace = 8 * N * (N + 1);   // the eight face slabs, rows padded like a block's pencils
    T s[Slab<N>::size];
    T t[kFace > Slab<N>::size ? kFace : Slab<N>::size];
};

// Face tables of the wave rows, with h0 = g0 / 2 (sign-flipped for the
// Hermite-type basis: g1 = -g0 reversed holds in both): c[1][t] = -h0[t]
// minus sigma at t = 0 weighs layer t (counted from the face) of a neighbour,
// c[0][t] = h0[t] the cell's own layers at a boundary face; he and ho are the
// even and odd halves of h0.
template <int N, typename T>
struct WaveFace {
    T c[2][N];
    T he[EOShape<N>::HC], ho[EOShape<N>::H];
};

// What two opposite faces add to a pencil, in its even and odd halves:
// E_i += he_i bd (+ ad at i = 0), O_i += ho_i bs (+ as at i = 0), with
// ad, as = (alpha_lower +- alpha_upper) / 2, bd, bs = beta_lower -+ beta_upper.
template <typename T>
struct FacePair {
    T ap, am, bd, bs;
    __device__ __forceinline__ FacePair(T al, T bl, T ah, T bh)
        : ap(T(0.5) * (al + ah)), am(T(0.5) * (al - ah)), bd(bl - bh), bs(bl + bh) {}
    __device__ __forceinline__ FacePair(const T* f, int st) : ap(f[0]), am(f[st]), bd(f[2 * st]), bs(f[3 * st]) {}
    template <int N>
    __device__ __forceinline__ void add(const WaveFace<N, T>& F, T s, T (&E)[EOShape<N>::HC],
                                        T (&O)[EOShape<N>::H]) const {
        const T sd = s * bd, ss = s * bs;
        E[0] = fma(s, ap, E[0]);
        O[0] = fma(s, am, O[0]);
#pragma unroll
        for (int i = 0; i < EOShape<N>::HC; ++i) E[i] = fma(F.he[i], sd, E[i]);
#pragma unroll
        for (int i = 0; i < EOShape<N>::H; ++i) O[i] = fma(F.ho[i], ss, O[i]);
    }
};

// lo = (a of the lower half-wave in lanes 0-31, b of it in lanes 32-63), hi =
// the same of the upper half-wave.
__device__ __forceinline__ void half_swap(double a, double b, double& lo, double& hi) {
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    lo = __hiloint2double(h[0], l[0]);
    hi = __hiloint2double(h[1], l[1]);
}

// The lane's x-pencil y[i] = (A u)_c at (i, j, k) with (j, k) = (pc.pa,
// pc.pb), for the active lanes; every lane of the wave must call it.
// TB: ME | MO | PE | PO (even-odd halves of M_hat and of the cell-diagonal
// P_hat).
// HERM: the Hermite-type basis.  The even-odd tables then hold the matrices
// conjugated by D = diag(hermite_sign) (centrosymmetric), so every value is
// multiplied by its sign s(i) s(j) s(k) on load and on store, and the face
// terms read only the two layers next to the face (the others carry no
// weight: eq. (hermite_traces_3d)).
template <int N, typename T, bool VP, bool HERM = false>
__device__ __forceinline__ void wave_sipg_cell(const T* __restrict__ u, const MeshArgs& G, const T* TB,
                                               const WaveFace<N, T>& F, int64_t c, WaveLds<N, T>& L,
                                               T (&y)[N]) {
    using SL = Slab<N>;
    using S = EOShape<N>;
    constexpr int N3 = N * N * N, HC = S::HC, H = S::H;
    constexpr int LV = HERM ? 2 : N;               // layers of a face's source that carry weight
    constexpr int FR = N + 1, FS = N * (N + 1);    // face slab strides: row, slab
    const T* ME = TB;
    const T* MO = TB + S::SE;
    const T* PE = TB + S::SE + S::SO;
    const T* PO = TB + 2 * S::SE + S::SO;
    const Pencil<N> pc(1);
    const int pa = pc.pa, pb = pc.pb, lane = threadIdx.x;
    // FP64 at n = 8: every lane is active, but the compiler must not know, so
    // that the phases stay separate blocks; merged, the scalar tables of all of
    // them are loaded ahead and spilled (48^3 cells: 310 us against 296)
    bool act = pc.act;
    if constexpr (Pencil<N>::kFull && sizeof(T) == 8) {
        int l = lane;
        asm("" : "+v"(l));
        act = l < 64;
    }
    const T* ub = u + G.offset;
    const int lb = G.logB;
    const uint32_t cu = static_cast<uint32_t>(c);
    const uint32_t cz = cu % static_cast<uint32_t>(G.mz);
    const uint32_t rr = cu / static_cast<uint32_t>(G.mz);
    const uint32_t cy = rr % static_cast<uint32_t>(G.my);
    const uint32_t cx = rr / static_cast<uint32_t>(G.my);
    const T sx = static_cast<T>(G.sx), sy = static_cast<T>(G.sy), sz = static_cast<T>(G.sz);
    const int64_t syz = static_cast<int64_t>(G.my) * G.mz;
    auto sg = [](int i) { return HERM ? static_cast<T>(hermite_sign(N, i)) : T(1); };
    const T sab = sg(pa) * sg(pb);   // sign of the lane's two tangential indices
    T* fs = L.t;
    // alpha and beta of one face from layers v_t counted from the source's
    // side of the face (rev: the source's last layer is next to the face)
    auto reduce = [&](const T (&v)[N], bool interior, bool rev, T& al, T& be) {
        const T* cf = F.c[interior ? 1 : 0];
        al = cf[0] * v[0];
#pragma unroll
        for (int t = 1; t < LV; ++t) al = fma(cf[t], v[t], al);
        be = rev ? -v[0] : v[0];
    };
    // lane (a, b) reads its pencil along the normal (stride ST)
    auto face = [&](auto STc, auto UPc, bool interior, int64_t d, T& al, T& be) {
        constexpr int ST = decltype(STc)::value;
        constexpr bool UP = decltype(UPc)::value;
        const bool rev = UP != interior;
        const int q0 = (ST == N * N ? pa * N + pb : ST == N ? pa * N * N + pb : (pa * N + pb) * N) +
                       (rev ? (N - 1) * ST : 0);
        const int step = rev ? -ST : ST;
        const T* p = ub + block_base(interior ? c + d : c, lb, N3) + (static_cast<int64_t>(q0) << lb);
        T v[N];
#pragma unroll
        for (int t = 0; t < LV; ++t) {
            v[t] = ldc<T>(p + (static_cast<int64_t>(t * step) << lb));
            // (layer t from the face: its sign is that of index t or N - 1 - t)
            if (HERM) v[t] *= sab * (rev ? sg(N - 1 - t) : sg(t));
        }
        reduce(v, interior, rev, al, be);
    };
    // The four slabs of one axis (normal stride ST) at o.  In FP64 at n = 8 a
    // lane takes two neighbouring pencils of one face (lanes 0-31 the lower,
    // 32-63 the upper face) with 16-byte loads, which the vector cache serves
    // at twice the rate of 8-byte ones, and a half-wave swap brings both faces
    // of a pencil together.
    constexpr bool kPairs = N == 8 && sizeof(T) == 8 && VP;
    auto axis = [&](auto STc, T* o, bool lo, bool hi, int64_t d) {
        constexpr int ST = decltype(STc)::value;
        T al, bl, ah, bh;
        int ra = pa, rb = pb;
        if constexpr (kPairs) {
            const bool up = lane >= 32;
            const int p = lane & 31, ca = p / (N / 2), cb = 2 * (p % (N / 2));
            const bool interior = up ? hi : lo, rev = up != interior;
            const int q0 = (ST == N * N ? ca * N + cb : ca * N * N + cb) + (rev ? (N - 1) * ST : 0);
            const int step = rev ? -ST : ST;
            const T* w = ub + block_base(interior ? c + (up ? d : -d) : c, 0, N3) + q0;
            typedef T Vec __attribute__((ext_vector_type(2)));
            Vec v[LV];
#pragma unroll
            for (int t = 0; t < LV; ++t) {
                v[t] = *reinterpret_cast<const Vec*>(w + t * step);
                if (HERM) {
                    const T s = sg(ca) * (rev ? sg(N - 1 - t) : sg(t));
                    v[t].x *= s * sg(cb), v[t].y *= s * sg(cb + 1);
                }
            }
            Vec va;
            auto weigh = [&](auto cf) {
                va = cf(0) * v[0];
#pragma unroll
                for (int t = 1; t < LV; ++t) va = Vec{fma(cf(t), v[t].x, va.x), fma(cf(t), v[t].y, va.y)};
            };
            // (uniform branches: scalar weights where both faces have the same)
            if (lo && hi) weigh([&](int t) { return F.c[1][t]; });
            else weigh([&](int t) { return interior ? F.c[1][t] : F.c[0][t]; });
            const Vec vb = rev ? -v[0] : v[0];
            half_swap(va.x, va.y, al, ah);
            half_swap(vb.x, vb.y, bl, bh);
            ra = ca, rb = cb + (up ? 1 : 0);
        } else {
            face(STc, std::integral_constant<bool, false>{}, lo, -d, al, bl);
            face(STc, std::integral_constant<bool, true>{}, hi, d, ah, bh);
        }
        const FacePair<T> f(al, bl, ah, bh);
        o += ra * FR + rb;
        o[0] = f.ap, o[FS] = f.am, o[2 * FS] = f.bd, o[3 * FS] = f.bs;
    };
    // The z neighbours' pencils come whole where 16-byte loads fetch them, and in
    // the Lagrange basis, which weighs every layer.  Else two layers of each are
    // enough: whole pencils took 2 n loads a lane more for nothing (28^3 cells at
    // B = 64, FP64, n = 6: 80 us against 68).
    constexpr bool kZLayers = HERM && !VP;
    const bool xl = cx > 0, xh = cx + 1 < static_cast<uint32_t>(G.mx);
    const bool yl = cy > 0, yh = cy + 1 < static_cast<uint32_t>(G.my);
    const bool zl = cz > 0, zh = cz + 1 < static_cast<uint32_t>(G.mz);
    T x[N], zal = T(0), zbl = T(0), zah = T(0), zbh = T(0);
    if (act) {
        const int64_t zp = static_cast<int64_t>((pa * N + pb) * N) << lb;
        pencil_load<N, VP>(x, ub + block_base(c, lb, N3) + zp, lb);
        T wl[N], wh[N];
        if constexpr (kZLayers) {
            face(std::integral_constant<int, 1>{}, std::integral_constant<bool, false>{}, zl, -1, zal, zbl);
            face(std::integral_constant<int, 1>{}, std::integral_constant<bool, true>{}, zh, 1, zah, zbh);
        } else {
            pencil_load<N, VP>(wl, ub + block_base(zl ? c - 1 : c, lb, N3) + zp, lb);
            pencil_load<N, VP>(wh, ub + block_base(zh ? c + 1 : c, lb, N3) + zp, lb);
        }
        axis(std::integral_constant<int, N>{}, fs, yl, yh, static_cast<int64_t>(G.mz));
        axis(std::integral_constant<int, N * N>{}, fs + 4 * FS, xl, xh, syz);
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (HERM) x[k] *= sab * sg(k);
        if constexpr (!kZLayers) {
            // z faces, layers counted from the face (lower: reversed when interior)
#pragma unroll
            for (int k = 0; k < N; ++k)
                if (HERM) wl[k] *= sab * sg(k), wh[k] *= sab * sg(k);
            T rl[N], rh[N];
#pragma unroll
            for (int t = 0; t < N; ++t) rl[t] = wl[N - 1 - t], rh[t] = wh[N - 1 - t];
            if constexpr (N == 8) {   // uniform branches; n = 5 and 6 are 4% faster with selects
                if (zl) reduce(rl, true, true, zal, zbl);
                else reduce(wl, false, false, zal, zbl);
                if (zh) reduce(wh, true, false, zah, zbh);
                else reduce(rh, false, true, zah, zbh);
            } else {
#pragma unroll
                for (int t = 0; t < N; ++t) rl[t] = zl ? rl[t] : wl[t], rh[t] = zh ? wh[t] : rh[t];
                reduce(rl, zl, zl, zal, zbl);
                reduce(rh, zh, !zh, zah, zbh);
            }
        }
    }
    wave_sync();
    auto mass_pencil = [&](T* p, int st) {
        T xin[N], e[HC], o[H], E[HC], O[H];
#pragma unroll
        for (int b = 0; b < N; ++b) xin[b] = p[b * st];
        eo_split<N>(xin, e, o);
        eo_mul<N>(ME, MO, e, o, E, O);
        eo_join<N>(E, O, xin);
#pragma unroll
        for (int b = 0; b < N; ++b) p[b * st] = xin[b];
    };
    // M_z on the rows of all eight slabs, M_y on the columns of the x slabs
    if (lane < 8 * N) mass_pencil(fs + (lane / N) * FS + (lane % N) * FR, 1);
    wave_sync();
    if (lane < 4 * N) mass_pencil(fs + (4 + lane / N) * FS + lane % N, FR);
    wave_sync();
    const FacePair<T> fy(fs + pa * FR + pb, FS), fx(fs + 4 * FS + pa * FR + pb, FS);
    wave_sync();
    T* A1 = L.t;
    T* A2 = L.s;
    if (act) {  // z: lane (i, j); t = M u, w = B_z u
        T e[HC], o[H], E[HC], O[H], r[N];
        eo_split<N>(x, e, o);
        eo_mul<N>(ME, MO, e, o, E, O);
        eo_join<N>(E, O, r);
#pragma unroll
        for (int k = 0; k < N; ++k) A1[SL::at(pa, pb, k)] = r[k];
        eo_mul<N>(PE, PO, e, o, E, O);
        FacePair<T>(zal, zbl, zah, zbh).template add<N>(F, T(1), E, O);
        eo_join<N>(E, O, r);
#pragma unroll
        for (int k = 0; k < N; ++k) A2[SL::at(pa, pb, k)] = r[k];
    }
    wave_sync();
    if (act) {  // y: lane (i, k); a = s_x M t, b = s_y B_y t + s_z M w
        T et[HC], ot[H], ew[HC], ow[H], E[HC], O[H], E2[HC], O2[H], r[N];
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = A1[SL::at(pa, j, pb)];
        eo_split<N>(r, et, ot);
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = A2[SL::at(pa, j, pb)];
        eo_split<N>(r, ew, ow);
        eo_mul<N>(ME, MO, et, ot, E, O);
        eo_join<N>(E, O, r);
#pragma unroll
        for (int j = 0; j < N; ++j) A1[SL::at(pa, j, pb)] = r[j] * sx;
        eo_mul<N>(PE, PO, et, ot, E, O);
        fy.template add<N>(F, T(1), E, O);
        eo_mul<N>(ME, MO, ew, ow, E2, O2);
#pragma unroll
        for (int i = 0; i < HC; ++i) E[i] = fma(sy, E[i], sz * E2[i]);
#pragma unroll
        for (int i = 0; i < H; ++i) O[i] = fma(sy, O[i], sz * O2[i]);
        eo_join<N>(E, O, r);
#pragma unroll
        for (int j = 0; j < N; ++j) A2[SL::at(pa, j, pb)] = r[j];
    }
    wave_sync();
    if (act) {  // x: lane (j, k); v = P a + M b and the x faces
        T ea[HC], oa[H], eb[HC], ob[H], E[HC], O[H], E2[HC], O2[H], r[N];
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = A1[SL::at(i, pa, pb)];
        eo_split<N>(r, ea, oa);
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = A2[SL::at(i, pa, pb)];
        eo_split<N>(r, eb, ob);
        eo_mul<N>(PE, PO, ea, oa, E, O);
        fx.template add<N>(F, sx, E, O);
        eo_mul<N>(ME, MO, eb, ob, E2, O2);
#pragma unroll
        for (int i = 0; i < HC; ++i) E[i] += E2[i];
#pragma unroll
        for (int i = 0; i < H; ++i) O[i] += O2[i];
        eo_join<N>(E, O, y);
        if (HERM) {
#pragma unroll
            for (int i = 0; i < N; ++i) y[i] *= sab * sg(i);
        }
    }
    wave_sync();
}

// The face tables of a plan's wave rows.
template <int N, typename T>
WaveFace<N, T> wave_face(const Plan& plan) {
    const RefData& ref = plan.ref[N];
    const bool herm = plan.basis == TP_BASIS_HERMITE;
    double h[N];
    for (int k = 0; k < N; ++k) h[k] = 0.5 * ref.g0[k] * (herm ? hermite_sign(N, k) : 1.0);
    WaveFace<N, T> F;
    for (int k = 0; k < N; ++k) {
        F.c[1][k] = static_cast<T>(-h[k] - (k == 0 ? plan.penalty_C * (N - 1) * N : 0.0));
        F.c[0][k] = static_cast<T>(h[k]);
    }
    for (int i = 0; i < EOShape<N>::H; ++i) {
        F.he[i] = static_cast<T>(0.5 * (h[i] + h[N - 1 - i]));
        F.ho[i] = static_cast<T>(0.5 * (h[i] - h[N - 1 - i]));
    }
    if constexpr (N % 2 == 1) F.he[N / 2] = static_cast<T>(h[N / 2]);
    return F;
}

}  // namespace tpfdm
