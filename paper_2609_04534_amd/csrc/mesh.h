// Parts shared by the kernels of a uniform box mesh: the mesh arguments, the
// 1D tables of the coupled SIPG operator, tile orders and the PCG state.
#pragma once

#include "device.h"

namespace tpfdm {

// Device-side state of a PCG solve (pcg.hip; the multigrid kernels of a
// solve read its done flag).  done: 0 running, 1 converged, 2 breakdown or
// a non-finite scalar, 3 iteration limit.
struct PcgState {
    double rz, pq, rr, bb, alpha, beta, tol2;
    int iter, done, maxit;
    int norm;   // stopping test on 0: (r, r), 1: (r, z) (tol2 scaled to match)
};

struct MeshArgs {
    int64_t ncells;
    int64_t offset;
    int logB;
    int mx, my, mz;
    double sx, sy, sz;   // s_d = h_o1 h_o2 / h_d
};

template <int N, typename T>
struct FaceRef {        // reference endpoint derivatives and penalty C p (p+1)
    T g0[N];
    T g1[N];
    T sigma;
};

// Tile of workgroup b on a mesh with about S tiles per x-plane of cells: each
// XCD walks its range in groups of SW consecutive tiles carried through the
// range's rows of S tiles.  A tile's x neighbours then come SW tiles apart in
// the visiting order instead of S, and are still in the XCD's L2 when the
// second of them reads them.  A bijection on [0, nwg): the last group of a
// row is S mod SW wide when SW does not divide S; the part of the range past
// its last whole row, and S = 0, keep the plain order.
__device__ __forceinline__ unsigned sweep_tile(unsigned b, unsigned nwg, unsigned S, unsigned SW) {
    const XcdRange x = xcd_range(b, nwg);
    const unsigned l = x.place;
    if (S == 0) return x.first + l;
    const unsigned R = x.count / S;
    if (R < 2 || l >= R * S) return x.first + l;
    const unsigned full = (S / SW) * SW * R;   // tiles in whole-width groups
    if (l < full) {
        const unsigned chunk = l / (SW * R), r = (l / SW) % R, g = l % SW;
        return x.first + r * S + chunk * SW + g;
    }
    const unsigned w = S % SW, e = l - full;          // w > 0 here
    return x.first + (e / w) * S + (S - w) + e % w;
}

// The tile kernels (n <= 4) sweep groups of 8 tiles.
constexpr unsigned kLaneSweep = 8;
__device__ __forceinline__ unsigned lane_tile(unsigned b, unsigned nwg, unsigned S) {
    return sweep_tile(b, nwg, S, kLaneSweep);
}

// The one-cell-per-wave kernels (n >= 5) sweep groups of 192 cells (n = 8 in
// FP64 on 48^3 cells: 317 us in plain order, 306, 296, 299 and 302 us with 48,
// 192, 384 and 768; FP32 within 4%, n = 6 within 1%).
// WV > 1 (workgroups of WV waves, one cell each): groups of as many cells.
template <int WV = 1>
__device__ __forceinline__ unsigned wave_tile(unsigned b, unsigned nwg, const MeshArgs& G) {
    return sweep_tile(b, nwg, static_cast<unsigned>(G.my) * static_cast<unsigned>(G.mz) / WV, 192 / WV);
}

// Row length S for lane_tile: the whole tiles of 64 W cells in an x-plane of
// cells when one plane of blocks (n^3 values of T per cell) holds 2 MiB or
// more, else 0 (plain order).  Coupled operator at n = 4, plain against
// grouped order: FP64 128^3 cells (8 MiB planes) 655 / 550 us, 100^3 346 /
// 300 us, 64^3 (2 MiB) 76 / 72 us; FP32 128^3 330 / 321 us; Hermite-type
// basis 128^3 478 / 453 us.  With an earlier form of the row groups of 4 to 32
// tiles differed by under 5%, and at n = 2 with 1 MiB planes the grouped order
// took 50 us against 46.
template <int N, typename T, int W>
__device__ __forceinline__ unsigned plane_tiles(const MeshArgs& G) {
    constexpr int64_t kMinPlaneBytes = int64_t(2) << 20;
    const int64_t p = static_cast<int64_t>(G.my) * G.mz;
    if (p * N * N * N * static_cast<int64_t>(sizeof(T)) < kMinPlaneBytes) return 0u;
    return static_cast<unsigned>(p / (64 * W));
}

// Kernel arguments of a mesh plan's group.
inline MeshArgs mesh_args(const Plan& plan, const GroupInfo& g) {
    MeshArgs G;
    G.ncells = g.nblocks;
    G.offset = g.offset;
    G.logB = g.logB;
    G.mx = plan.mesh_m[0];
    G.my = plan.mesh_m[1];
    G.mz = plan.mesh_m[2];
    const double hx = plan.mesh_h[0], hy = plan.mesh_h[1], hz = plan.mesh_h[2];
    G.sx = hy * hz / hx;
    G.sy = hx * hz / hy;
    G.sz = hx * hy / hz;
    return G;
}

// 1D tables of the coupled operator: M_hat and the cell-diagonal P_hat
// (A_hat, or A_hat - K_hat for the face part alone), endpoint derivatives and
// the reference penalty.
template <int N, typename TC>
void sipg_tables(const Plan& plan, bool face_only, Pair<N, TC>& R, FaceRef<N, TC>& F) {
    const RefData& ref = plan.ref[N];
    for (int i = 0; i < N * N; ++i) {
        R.m[i] = static_cast<TC>(ref.M[i]);
        R.p[i] = static_cast<TC>(face_only ? ref.A[i] - ref.K[i] : ref.A[i]);
    }
    for (int i = 0; i < N; ++i) {
        F.g0[i] = static_cast<TC>(ref.g0[i]);
        F.g1[i] = static_cast<TC>(ref.g1[i]);
    }
    F.sigma = static_cast<TC>(plan.penalty_C * (N - 1) * N);
}

}  // namespace tpfdm
