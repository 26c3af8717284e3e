// Geometric multigrid for the coupled SIPG operator of a mesh plan (n <= 8):
// the V-cycle the paper uses to precondition CG (Sec. 5, Sec. 6.1).
//
// Levels: the plan's box and its uniform coarsenings (cells halved in every
// direction while all three counts are even, cell lengths doubled, the
// operator rediscretized with the level's own lengths and penalty).  On each
// level but the coarsest one smoothing application before and one after
// the coarse correction; a smoothing application is the degree-three
// Chebyshev-accelerated block-Jacobi method, three Richardson updates
//   u <- u + omega_j D^{-1} (b - A u),  omega_j = 1 / (c - d cos((2j-1) pi / 6))
// on the spectral interval [0.2, 2] (eq. (chebyshev_weights),
// eq. (chebyshev_richardson)), with D^{-1} the cell-wise fast-diagonalization
// inverse.  All tables (operator, inverse, transfers) are the plan's, in the
// plan's basis.  Each update is one kernel in the factorized form the paper
// describes (Sec. 5.2): the operator row, the residual, the block inverse
// and the update of a workgroup's cells in registers and LDS, so no residual
// vector is written; the first update from u = 0 needs no operator.  Updates alternate
// between the correction and one scratch vector per level.  Transfers embed
// a coarse cell's polynomial into its eight children (prolongation, added
// to the fine correction) and apply the transpose (restriction).  The coarsest level is solved exactly by a
// dense inverse, assembled once by applying the level operator to unit
// vectors (as the paper assembles its coarse LU) and inverted on the host.
//
// For n <= 4 every vector of a level is in the B = 64 blocked layout, 64 or 128
// cells per workgroup of n waves (a wave holds a plane of each cell); for n >= 5
// in the B = 1 layout, one cell per wave.  Every kernel returns at once when the
// solve state passed to it is done, so a V-cycle can sit inside captured CG
// iterations.
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <new>
#include <thread>
#include <tuple>
#include <type_traits>
#include <vector>

#include "sipg.h"

namespace tpfdm {

constexpr int64_t kMaxCoarse = 2048;   // unknowns of the densely solved coarsest level

template <int N>
struct ProlTab {    // 1D embeddings of the left and right child, row-major
    double p[2][N * N];
};

namespace {

__device__ __forceinline__ bool done_flag(const PcgState* st) { return st && st->done; }

// Level vectors are stored in TS (double, or float for the FP32-storage
// hierarchy).  The operator rows of the smoother and of the residual are
// computed in MgTC<TS>: FP64 for FP64 storage, FP32 for FP32 storage (there
// the level vectors carry FP32 rounding already, and the FP32 rows take half
// the registers and LDS of FP64 ones); the smoother's block inverse runs in
// TI, the updates u + omega D^{-1} r and the transfers in FP64, and every kernel
// rounds only where it stores.
template <typename TS>
using MgTC = typename std::conditional<std::is_same<TS, float>::value, float, double>::type;

// t = A u on one level (64 W cells per workgroup of N waves); the consumers
// form b - t as they load.
template <int N, bool HERM, typename TS, int W = 1>
__global__ __launch_bounds__(64 * N, (tile_waves<N, MgTC<TS>, W>())) void k_mg_apply(
    const TS* __restrict__ u, TS* __restrict__ t, MeshArgs G, TileTab<N, MgTC<TS>, HERM> R,
    const PcgState* __restrict__ st) {
    using TC = MgTC<TS>;
    if (done_flag(st)) return;
    constexpr int N2 = N * N, N3 = N * N * N;
    __shared__ Cells<TC, W> A[N3][64];
    const TileCell<W> T(G, lane_tile(blockIdx.x, gridDim.x, plane_tiles<N, TS, W>(G)));
    Cells<TC, W> out[N2];
    tile_sipg<N, TS, TC, W, 6, HERM>(u, G, R, T, A, out);
    if (!T.valid) return;
    TS* tb = t + G.offset + block_base(T.c, 6, N3) + (static_cast<int64_t>(T.w * N2) << 6);
#pragma unroll
    for (int e = 0; e < N2; ++e) st_cells<false>(tb + (e << 6), out[e]);
}

// u = omega D^{-1} b: the first Chebyshev update from u = 0 (no operator
// application), the block inverse in precision TI, its weight in FP64.
template <int N, typename TI, typename TS>
__global__ __launch_bounds__(64 * N, 4) void k_mg_jacobi0(const TS* __restrict__ b, TS* __restrict__ u, MeshArgs G,
                                                          TileInv<N, TI> E, double omega,
                                                          const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    constexpr int N2 = N * N, N3 = N * N * N;
    __shared__ Cells<TI, 1> A[N3][64];
    const TileCell<1> T(G, blockIdx.x);
    const int64_t base = G.offset + block_base(T.c, 6, N3) + (static_cast<int64_t>(T.w * N2) << 6);
    Cells<TI, 1> v[N2];
#pragma unroll
    for (int e = 0; e < N2; ++e) v[e].v[0] = static_cast<TI>(b[base + (e << 6)]);
    tile_fdm<N, TI, 1>(E, T, A, v);
    if (!T.valid) return;
#pragma unroll
    for (int e = 0; e < N2; ++e) u[base + (e << 6)] = static_cast<TS>(omega * static_cast<double>(v[e].v[0]));
}

// One Chebyshev update in a single pass (the factorized form: no residual
// vector is stored): u_out = u_in + omega D^{-1} (b - A u_in) for the
// workgroup's cells, A u_in from the cells and their six neighbours, the block
// inverse in precision TI on the residual planes, the update in FP64.  u_out must
// not alias u_in (other workgroups still read u_in).
// DOT: also a partial of (r, u_out) per workgroup, for CG: r is read once more
// here (64^3 cells, n = 4, FP64: 116 -> 132 us), where a kernel of its own read
// both vectors (46 us).
template <int N, typename TI, bool HERM, typename TS, int W = 1, bool DOT = false>
__global__ __launch_bounds__(64 * N, (tile_waves<N, MgTC<TS>, W>())) void k_mg_smooth(
    const TS* __restrict__ b, const TS* __restrict__ uin, TS* __restrict__ uout, MeshArgs G, TileTab<N, MgTC<TS>, HERM> R,
    TileInv<N, TI> E, double omega, const PcgState* __restrict__ st, const double* __restrict__ r,
    double* __restrict__ part) {
    using TC = MgTC<TS>;
    if (done_flag(st)) return;
    constexpr int N2 = N * N, N3 = N * N * N;
    constexpr size_t kBytes = N3 * 64 * W * (sizeof(TC) > sizeof(TI) ? sizeof(TC) : sizeof(TI));
    __shared__ __align__(16) char lds[kBytes];
    const TileCell<W> T(G, lane_tile(blockIdx.x, gridDim.x, plane_tiles<N, TS, W>(G)));
    Cells<TC, W> out[N2];
    tile_sipg<N, TS, TC, W, 6, HERM>(uin, G, R, T, reinterpret_cast<Cells<TC, W>(*)[64]>(lds), out);
    const int64_t base = G.offset + block_base(T.c, 6, N3) + (static_cast<int64_t>(T.w * N2) << 6);
    Cells<TI, W> v[N2];
#pragma unroll
    for (int e = 0; e < N2; ++e) {
        const Cells<TC, W> bv = ld_cells<TC, W>(b + base + (e << 6));
#pragma unroll
        for (int k = 0; k < W; ++k) v[e].v[k] = static_cast<TI>(bv.v[k] - out[e].v[k]);
    }
    // the planes of the two element types do not coincide
    if constexpr (sizeof(TC) != sizeof(TI)) tile_sync();
    tile_fdm<N, TI, W>(E, T, reinterpret_cast<Cells<TI, W>(*)[64]>(lds), v);
    double s = 0.0;
    if (T.valid) {
#pragma unroll
        for (int e = 0; e < N2; ++e) {
            Cells<double, W> uv = ld_cells<double, W>(uin + base + (e << 6));
#pragma unroll
            for (int k = 0; k < W; ++k) uv.v[k] = ::fma(omega, static_cast<double>(v[e].v[k]), uv.v[k]);
            st_cells<false>(uout + base + (e << 6), uv);
            if constexpr (DOT) {
                const Cells<double, W> rv = ld_cells<double, W>(r + base + (e << 6));
#pragma unroll
                for (int k = 0; k < W; ++k) s = fma(rv.v[k], static_cast<double>(static_cast<TS>(uv.v[k])), s);
            }
        }
    }
    if constexpr (DOT) {
        tile_sync();
        s = tile_sum<N>(s, reinterpret_cast<double*>(lds));
        if (threadIdx.x == 0 && threadIdx.y == 0) part[blockIdx.x] = s;
    }
}

// The child's 1D embedding (or its transpose) of a lane's cell along an axis.
template <int N>
__device__ __forceinline__ void child_matrix(const ProlTab<N>& P, bool upper, double (&m)[N * N]) {
#pragma unroll
    for (int e = 0; e < N * N; ++e) m[e] = upper ? P.p[1][e] : P.p[0][e];
}

// v <- (X (x) Y (x) Z) v for the lane's cell, each factor the embedding P of
// the cell's half along that axis (ux, uy, uz: upper); v the plane i = w in
// and out, the x contraction through LDS.  A: N^3 x 64 doubles whose plane
// i = w the wave owns on entry and on return.
template <int N>
__device__ __forceinline__ void tile_kron(const ProlTab<N>& P, bool ux, bool uy, bool uz, int w, int lane,
                                          double (*A)[64], double (&v)[N * N]) {
    constexpr int N2 = N * N;
    auto pencil = [&](const double (&m)[N2], double (&x)[N2], int base, int st) {
        double t[N];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            t[r] = m[r * N] * x[base];
#pragma unroll
            for (int k = 1; k < N; ++k) t[r] = fma(m[r * N + k], x[base + k * st], t[r]);
        }
#pragma unroll
        for (int r = 0; r < N; ++r) x[base + r * st] = t[r];
    };
    double m[N2];
    child_matrix<N>(P, uz, m);
#pragma unroll
    for (int jj = 0; jj < N; ++jj) pencil(m, v, jj * N, 1);
    child_matrix<N>(P, uy, m);
#pragma unroll
    for (int k = 0; k < N; ++k) pencil(m, v, k, N);
#pragma unroll
    for (int q = 0; q < N2; ++q) A[w * N2 + q][lane] = v[q];
    tile_sync();
    child_matrix<N>(P, ux, m);
    double x[N2];   // x-z plane j = w
#pragma unroll
    for (int l = 0; l < N; ++l)
#pragma unroll
        for (int k = 0; k < N; ++k) x[l * N + k] = A[(l * N + w) * N + k][lane];
#pragma unroll
    for (int k = 0; k < N; ++k) pencil(m, x, k, N);
#pragma unroll
    for (int l = 0; l < N; ++l)
#pragma unroll
        for (int k = 0; k < N; ++k) A[(l * N + w) * N + k][lane] = x[l * N + k];
    tile_sync();
#pragma unroll
    for (int q = 0; q < N2; ++q) v[q] = A[w * N2 + q][lane];
}

// b_coarse = P^T (b_fine - t_fine), t_fine = A u_fine: 64 coarse cells per
// workgroup of 2 N waves, wave (w, bx) on the y-z planes i = w of the children
// in x half bx.  The z pair of children are consecutive cells: one access of
// two values a lane loads both.  Contractions along z and y run on the loaded
// planes, the one along x through LDS into the x-z plane j = w, half of its
// rows per wave.  (One coarse cell a lane, all eight children in turn, took 87
// us on 32^3 coarse cells at n = 4 and 21-25 us on any smaller level.)
template <int N, typename TS>
__global__ __launch_bounds__(128 * N) void k_mg_restrict(const TS* __restrict__ bf, const TS* __restrict__ tf,
                                                         TS* __restrict__ bc, MeshArgs Gf, MeshArgs Gc,
                                                         ProlTab<N> PT, const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    constexpr int N2 = N * N, N3 = N * N * N;
    __shared__ double A[2][N3][64];
    const TileCell<1> T(Gc, blockIdx.x);
    const int w = T.w % N, bx = T.w / N, lane = T.lane;
    // (two values aligned to one: the caller's right-hand side may be)
    typedef TS Vec __attribute__((ext_vector_type(2), aligned(sizeof(TS))));
    double acc[N2];
#pragma unroll
    for (int by = 0; by < 2; ++by) {
        const int64_t f = (static_cast<int64_t>(2 * T.cx + bx) * Gf.my + (2 * T.cy + by)) * Gf.mz + 2 * T.cz;
        const int64_t o = Gf.offset + block_base(f, 6, N3) + (static_cast<int64_t>(w * N2) << 6);
        double t[N2];
#pragma unroll
        for (int jj = 0; jj < N; ++jj) {
            double r[2][N];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const Vec bv = *reinterpret_cast<const Vec*>(bf + o + ((jj * N + k) << 6));
                const Vec tv = *reinterpret_cast<const Vec*>(tf + o + ((jj * N + k) << 6));
#pragma unroll
                for (int bz = 0; bz < 2; ++bz) r[bz][k] = static_cast<double>(bv[bz]) - static_cast<double>(tv[bz]);
            }
#pragma unroll
            for (int k = 0; k < N; ++k) {
                double s = 0.0;
#pragma unroll
                for (int bz = 0; bz < 2; ++bz)
#pragma unroll
                    for (int kk = 0; kk < N; ++kk) s = fma(PT.p[bz][k * N + kk], r[bz][kk], s);
                t[jj * N + k] = s;
            }
        }
#pragma unroll
        for (int jj = 0; jj < N; ++jj)
#pragma unroll
            for (int k = 0; k < N; ++k) {
                double s = by == 0 ? 0.0 : acc[jj * N + k];
#pragma unroll
                for (int l = 0; l < N; ++l) s = fma(PT.p[by][jj * N + l], t[l * N + k], s);
                acc[jj * N + k] = s;
            }
    }
#pragma unroll
    for (int q = 0; q < N2; ++q) A[bx][w * N2 + q][lane] = acc[q];
    tile_sync();
    if (!T.valid) return;
    TS* o = bc + Gc.offset + block_base(T.c, 6, N3);
    constexpr int NH = (N + 1) / 2;   // rows of the first wave of a plane
#pragma unroll
    for (int k = 0; k < N; ++k) {
        double v[2][N];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int l = 0; l < N; ++l) v[b][l] = A[b][(l * N + w) * N + k][lane];
#pragma unroll
        for (int ii = 0; ii < NH; ++ii) {
            const int i = bx * NH + ii;
            if (i >= N) break;
            double s = 0.0;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int l = 0; l < N; ++l) s = fma(PT.p[b][i * N + l], v[b][l], s);
            o[((i * N + w) * N + k) << 6] = static_cast<TS>(s);
        }
    }
}

// u_out = u_fine + P u_coarse: 64 fine cells per workgroup of N waves, the
// child's embedding selected per lane.
template <int N, typename TS>
__global__ __launch_bounds__(64 * N, N == 4 ? 3 : 4) void k_mg_prolong(const TS* __restrict__ uc, const TS* __restrict__ uf,
                                                          TS* __restrict__ uout, MeshArgs Gf, MeshArgs Gc,
                                                          ProlTab<N> P, const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    constexpr int N2 = N * N, N3 = N * N * N;
    __shared__ double A[N3][64];
    const TileCell<1> T(Gf, blockIdx.x);
    const int64_t c = (static_cast<int64_t>(T.cx / 2) * Gc.my + T.cy / 2) * Gc.mz + T.cz / 2;
    const TS* wc = uc + Gc.offset + block_base(c, 6, N3) + (static_cast<int64_t>(T.w * N2) << 6);
    const int64_t o = Gf.offset + block_base(T.c, 6, N3) + (static_cast<int64_t>(T.w * N2) << 6);
    double v[N2], uv[N2];
#pragma unroll
    for (int q = 0; q < N2; ++q) v[q] = static_cast<double>(wc[q << 6]);
#pragma unroll
    for (int q = 0; q < N2; ++q) uv[q] = static_cast<double>(uf[o + (q << 6)]);
    tile_kron<N>(P, T.cx & 1, T.cy & 1, T.cz & 1, T.w, T.lane, A, v);
    if (!T.valid) return;
#pragma unroll
    for (int q = 0; q < N2; ++q) uout[o + (q << 6)] = static_cast<TS>(uv[q] + v[q]);
}

// u = A0^{-1} b on the coarsest level: one row of the (symmetric) inverse per
// wave, its dot product with b spread over the lanes.  (One row per thread, a
// chain of n0 dependent loads, took 28 us at n0 = 216.)
constexpr int kCoarseRows = 4;   // rows (waves) per workgroup
template <int N, typename TS>
__global__ __launch_bounds__(64 * kCoarseRows) void k_mg_coarse(const double* __restrict__ inv,
                                                                const TS* __restrict__ b, TS* __restrict__ u, int n0,
                                                                int64_t offset, int lb,
                                                                const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    constexpr int N3 = N * N * N;
    const int row = blockIdx.x * kCoarseRows + threadIdx.y;
    if (row >= n0) return;
    auto pos = [&](int e) { return offset + block_base(e / N3, lb, N3) + (static_cast<int64_t>(e % N3) << lb); };
    const double* a = inv + static_cast<int64_t>(row) * n0;
    double s = 0.0;
#pragma unroll 4
    for (int j = threadIdx.x; j < n0; j += 64) s = fma(a[j], static_cast<double>(b[pos(j)]), s);
    s = wave_sum(s);
    if (threadIdx.x == 0) u[pos(row)] = static_cast<TS>(s);
}
inline unsigned coarse_grid(int64_t n0) { return static_cast<unsigned>((n0 + kCoarseRows - 1) / kCoarseRows); }

// The V-cycle below and including a level of at most 64 cells (n <= 4) in one
// workgroup of N waves with every level vector but the entry level's
// right-hand side in LDS.  On such levels a launch per step is all latency:
// 19 launches of 5-10 us each for 4^3, 2^3 and one cell against one of 52 us
// at n = 3 in FP32 and 117 us at n = 4 in FP64.
// Levels hold at most 64, 8 and 1 cells; all vectors are [q][64 lanes], the
// second and third level's at lane offsets of one shared block.
constexpr int kTailLevels = 3;
constexpr int kTailUnknowns = 256;   // of the coarsest level: its inverse is read by one CU
template <int N, typename TI, bool HERM, typename TS>
struct TailArgs {
    int levels;                       // 2 or 3, the coarsest included
    int n0;                           // unknowns of the coarsest level
    MeshArgs G[kTailLevels];
    TileTab<N, MgTC<TS>, HERM> R;
    TileInv<N, TI> E[kTailLevels - 1];
    ProlTab<N> P, PT;
    double omega[3];
    const double* inv;
};
template <int N, typename TI, bool HERM, typename TS>
__global__ __launch_bounds__(64 * N, 1) void k_mg_tail(const TS* __restrict__ b0, TS* __restrict__ u0,
                                                       TailArgs<N, TI, HERM, TS> M, const PcgState* __restrict__ st) {
    using TC = MgTC<TS>;
    if (done_flag(st)) return;
    constexpr int N2 = N * N, N3 = N * N * N;
    __shared__ TS ua[N3 * 64], ta[N3 * 64], lower[N3 * 64];
    __shared__ double A[N3][64];
    TC(*At)[64] = reinterpret_cast<TC(*)[64]>(&A[0][0]);
    TI(*Ai)[64] = reinterpret_cast<TI(*)[64]>(&A[0][0]);
    const int lane = threadIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    // correction, scratch and right-hand side of a level
    auto u_of = [&](int l) { return l == 0 ? ua : lower + (l == 1 ? 0 : 24); };
    auto t_of = [&](int l) { return l == 0 ? ta : lower + 8; };
    auto b_of = [&](int l) { return lower + (l == 1 ? 16 : 25); };
    // own plane of the right-hand side (the entry level's is in global memory)
    auto rhs = [&](int l, const TileCell<1>& T, int q) {
        return l == 0 ? b0[((T.w * N2 + q) << 6) + T.c] : b_of(l)[((T.w * N2 + q) << 6) + T.c];
    };
    // one update u_to = u_from + omega D^{-1} (b - A u_from), or from zero
    auto update = [&](int l, const TS* from, TS* to, double omega) {
        const TileCell<1> T(M.G[l], 0);
        TI v[N2];
        Cells<TI, 1> vi[N2];
#pragma unroll
        for (int q = 0; q < N2; ++q) v[q] = static_cast<TI>(static_cast<TC>(rhs(l, T, q)));
        if (from) {
            Cells<TC, 1> out[N2];
            tile_sipg<N, TS, TC, 1, 6, HERM>(from, M.G[l], M.R, T, reinterpret_cast<Cells<TC, 1>(*)[64]>(At), out);
#pragma unroll
            for (int q = 0; q < N2; ++q) v[q] = static_cast<TI>(static_cast<TC>(rhs(l, T, q)) - out[q].v[0]);
            if constexpr (sizeof(TC) != sizeof(TI)) tile_sync();
        }
#pragma unroll
        for (int q = 0; q < N2; ++q) vi[q].v[0] = v[q];
        tile_fdm<N, TI, 1>(M.E[l], T, reinterpret_cast<Cells<TI, 1>(*)[64]>(Ai), vi);
        if (T.valid) {
#pragma unroll
            for (int q = 0; q < N2; ++q) {
                const int o = ((w * N2 + q) << 6) + lane;
                const double uv = from ? static_cast<double>(from[o]) : 0.0;
                to[o] = static_cast<TS>(fma(omega, static_cast<double>(vi[q].v[0]), uv));
            }
        }
        tile_sync();
    };
    const int last = M.levels - 1;
#pragma unroll 1
    for (int l = 0; l < last; ++l) {
        TS* u = u_of(l);
        TS* t = t_of(l);
        update(l, nullptr, u, M.omega[0]);
#pragma unroll 1
        for (int j = 1; j < 3; ++j) update(l, j == 1 ? u : t, j == 1 ? t : u, M.omega[j]);
        // residual, each child's part of the restriction, sums over children
        const TileCell<1> T(M.G[l], 0);
        Cells<TC, 1> out[N2];
        tile_sipg<N, TS, TC, 1, 6, HERM>(u, M.G[l], M.R, T, reinterpret_cast<Cells<TC, 1>(*)[64]>(At), out);
        tile_sync();
        double v[N2];
#pragma unroll
        for (int q = 0; q < N2; ++q)
            v[q] = static_cast<double>(rhs(l, T, q)) - static_cast<double>(static_cast<TS>(out[q].v[0]));
        tile_kron<N>(M.PT, T.cx & 1, T.cy & 1, T.cz & 1, w, lane, A, v);
        tile_sync();
        const MeshArgs& Gf = M.G[l];
        const MeshArgs& Gc = M.G[l + 1];
        TS* bc = b_of(l + 1);
        const int nc = static_cast<int>(Gc.ncells);
        for (int e = w * 64 + lane; e < N3 * nc; e += 64 * N) {
            const int q = e / nc, c = e - q * nc;
            const int cz = c % Gc.mz, cy = (c / Gc.mz) % Gc.my, cx = c / (Gc.mz * Gc.my);
            double s = 0.0;
#pragma unroll
            for (int ch = 0; ch < 8; ++ch)
                s += A[q][((2 * cx + (ch >> 2)) * Gf.my + 2 * cy + ((ch >> 1) & 1)) * Gf.mz + 2 * cz + (ch & 1)];
            bc[(q << 6) + c] = static_cast<TS>(s);
        }
        tile_sync();
    }
    {   // dense solve of the coarsest level: rows over lanes, columns over waves
        const TS* b = b_of(last);
        TS* u = u_of(last);
        double* part = &A[0][0];
        const int n0 = M.n0, j0 = w * n0 / N, j1 = (w + 1) * n0 / N;
        auto pos = [&](int e) { return ((e % N3) << 6) + e / N3; };
        for (int r = lane; r < n0; r += 64) {
            double s = 0.0;
#pragma unroll 8
            for (int j = j0; j < j1; ++j) s = fma(M.inv[static_cast<int64_t>(j) * n0 + r], static_cast<double>(b[pos(j)]), s);
            part[w * kTailUnknowns + r] = s;
        }
        tile_sync();
        for (int r = w * 64 + lane; r < n0; r += 64 * N) {
            double s = part[r];
#pragma unroll
            for (int k = 1; k < N; ++k) s += part[k * kTailUnknowns + r];
            u[pos(r)] = static_cast<TS>(s);
        }
        tile_sync();
    }
#pragma unroll 1
    for (int l = last - 1; l >= 0; --l) {
        TS* u = u_of(l);
        TS* t = t_of(l);
        const TileCell<1> T(M.G[l], 0);
        const MeshArgs& Gc = M.G[l + 1];
        const TS* uc = u_of(l + 1) + (T.cx / 2 * Gc.my + T.cy / 2) * Gc.mz + T.cz / 2;
        double v[N2];
#pragma unroll
        for (int q = 0; q < N2; ++q) v[q] = static_cast<double>(uc[(w * N2 + q) << 6]);
        tile_kron<N>(M.P, T.cx & 1, T.cy & 1, T.cz & 1, w, lane, A, v);
        if (T.valid) {
#pragma unroll
            for (int q = 0; q < N2; ++q) {
                const int o = ((w * N2 + q) << 6) + lane;
                t[o] = static_cast<TS>(static_cast<double>(u[o]) + v[q]);
            }
        }
        tile_sync();
#pragma unroll 1
        for (int j = 0; j < 3; ++j) update(l, j == 1 ? u : t, j == 1 ? t : u, M.omega[j]);
    }
    const TileCell<1> T(M.G[0], 0);
    if (T.valid) {
#pragma unroll
        for (int q = 0; q < N2; ++q) u0[((w * N2 + q) << 6) + lane] = ua[((w * N2 + q) << 6) + lane];
    }
}

// Partial (a, b) per 64-cell tile (the layout of the PCG partials).
template <int N, typename TS>
__global__ __launch_bounds__(64) void k_mg_dot(const double* __restrict__ a, const TS* __restrict__ b,
                                               MeshArgs G, double* __restrict__ part,
                                               const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    constexpr int N3 = N * N * N;
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x;
    double s = 0.0;
    if (c < G.ncells) {
        const int64_t base = G.offset + block_base(c, 6, N3);
#pragma unroll
        for (int e = 0; e < N3; ++e) {
            const int64_t o = base + (static_cast<int64_t>(e) << 6);
            s = fma(a[o], static_cast<double>(b[o]), s);
        }
    }
    s = wave_sum(s);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// ---------------------------------------------------------------- n >= 5
// One cell per wave (layout B = 1, FP64 or FP32 level vectors; the
// operator rows in the storage type, the transfers in FP64): lane (a, b) owns
// the z-pencil (a, b, 0..n-1) of the cell for loads and stores; the
// operator row is the wave body of the coupled operator (wave_sipg_cell,
// output by x-pencils), the block inverse the even-odd fast
// diagonalization in an LDS slab, and the transfers three 1D contractions
// through an LDS slab.

// Pencil base of lane (pa, pb)'s z-pencil of cell c.
template <int N>
__device__ __forceinline__ int64_t zpencil_base(const MeshArgs& G, int64_t c, const Pencil<N>& pc) {
    return G.offset + block_base(c, G.logB, N * N * N) + (static_cast<int64_t>((pc.pa * N + pc.pb) * N) << G.logB);
}

// The even-odd tables of a wave operator row: FP64 ones are read where they
// are used at wave-uniform global addresses (scalar loads), FP32 ones are
// loaded into registers once.
template <typename T, int TAB>
__device__ __forceinline__ const T* wave_row_tables(T (&regs)[sizeof(T) == 8 ? 1 : TAB], const T* tab) {
    if constexpr (sizeof(T) == 8) {
        return tab;
    } else {
        load_table<T, TAB>(regs, tab, nullptr);
        return regs;
    }
}

// t = A u, one cell per wave; the row in the level storage type T.
template <int N, bool VP, typename T = double>
__global__ __launch_bounds__(64, 2) void k_mg_apply_wave(const T* __restrict__ u, T* __restrict__ t,
                                                       MeshArgs G, const T* __restrict__ tab,
                                                       WaveFace<N, T> F, const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    constexpr int TAB = 2 * (EOShape<N>::SE + EOShape<N>::SO);
    __shared__ WaveLds<N, T> L;
    T regs[sizeof(T) == 8 ? 1 : TAB];
    const T* tb = wave_row_tables<T, TAB>(regs, tab);
    const int64_t c = wave_tile(blockIdx.x, gridDim.x, G);
    T y[N];
    wave_sipg_cell<N, T, VP, false>(u, G, tb, F, c, L, y);
    const Pencil<N> pc(1);
    if (pc.act) {
        T* out = t + G.offset + block_base(c, G.logB, N * N * N);
#pragma unroll
        for (int i = 0; i < N; ++i) out[static_cast<int64_t>((i * N + pc.pa) * N + pc.pb) << G.logB] = y[i];
    }
}

// z-pencil in, z = omega D^{-1} r of the wave's cell in precision TI in the
// slab, the lane's z-pencil of it returned (every lane of the wave calls it).
template <int N, typename TI>
__device__ __forceinline__ void wave_block_inverse(const Pencil<N>& pc, TI* slab, const TI* T, const TI* lam,
                                                   const MeshArgs& G, double (&r)[N]) {
    using SL = Slab<N>;
    eo_inverse_lds<N, TI>(pc, slab, T, T + EOShape<N>::SE, lam, static_cast<TI>(G.sx), static_cast<TI>(G.sy),
                          static_cast<TI>(G.sz));
    if (pc.act)
#pragma unroll
        for (int k = 0; k < N; ++k) r[k] = static_cast<double>(slab[SL::at(pc.pa, pc.pb, k)]);
}

// u = omega D^{-1} b (the first Chebyshev update from u = 0), one cell per wave.
template <int N, typename TI, bool VP, typename TS = double>
__global__ __launch_bounds__(64, 2) void k_mg_jacobi0_wave(const TS* __restrict__ b, TS* __restrict__ u,
                                                         MeshArgs G, const TI* __restrict__ tabS, double omega,
                                                         const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    using SL = Slab<N>;
    constexpr int TABM = EOShape<N>::SE + EOShape<N>::SO;
    __shared__ TI slab[SL::size];
    __shared__ TI stab[TABM + N];
    for (int e = threadIdx.x; e < TABM + N; e += 64) stab[e] = tabS[e];
    const int64_t c = blockIdx.x;
    const Pencil<N> pc(1);
    const int64_t pb = zpencil_base<N>(G, c, pc);
    double v[N];
    if (pc.act) {
        pencil_load<N, VP>(v, b + pb, G.logB);
#pragma unroll
        for (int k = 0; k < N; ++k) slab[SL::at(pc.pa, pc.pb, k)] = static_cast<TI>(v[k]);
    }
    wave_sync();
    wave_block_inverse<N, TI>(pc, slab, stab, stab + TABM, G, v);
    if (pc.act) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] *= omega;
        pencil_store<N, VP>(u + pb, v, G.logB);
    }
}

// One Chebyshev update u_out = u_in + omega D^{-1} (b - A u_in) of the
// wave's cell: the operator row by x-pencils, the residual into the slab in
// precision TI, the block inverse, the update by z-pencils.
template <int N, typename TI, bool VP, typename T = double, bool DOT = false>
__global__ __launch_bounds__(64, 2) void k_mg_smooth_wave(const T* __restrict__ b,
                                                        const T* __restrict__ uin, T* __restrict__ uout,
                                                        MeshArgs G, const T* __restrict__ tab,
                                                        WaveFace<N, T> F, const TI* __restrict__ tabS,
                                                        double omega, const PcgState* __restrict__ st,
                                                        const double* __restrict__ r, double* __restrict__ part) {
    if (done_flag(st)) return;
    using SL = Slab<N>;
    constexpr int TAB = 2 * (EOShape<N>::SE + EOShape<N>::SO);
    constexpr int TABM = EOShape<N>::SE + EOShape<N>::SO;
    __shared__ __align__(16) WaveLds<N, T> L;
    // the inverse's slab: the face scratch when it fits there, else the
    // whole (by then free) operator scratch, block slab included
    constexpr bool kInT = SL::size * sizeof(TI) <= sizeof(WaveLds<N, T>::t);
    static_assert(SL::size * sizeof(TI) <= sizeof(WaveLds<N, T>), "slab exceeds the operator scratch");
    __shared__ TI stab[TABM + N];
    for (int e = threadIdx.x; e < TABM + N; e += 64) stab[e] = tabS[e];
    T regs[sizeof(T) == 8 ? 1 : TAB];
    const T* tb = wave_row_tables<T, TAB>(regs, tab);
    const int64_t c = wave_tile(blockIdx.x, gridDim.x, G);
    const Pencil<N> pc(1);
    const T* bb = b + G.offset + block_base(c, G.logB, N * N * N);
    // FP32: the lane's x-pencil of b and z-pencil of u_in are loaded before
    // the operator row, so that their latency overlaps it (measured at p = 7
    // on 48^3 cells: MG-PCG 84.8 -> 74.8 ms, at five waves per SIMD instead
    // of seven); in FP64 the 32 more registers cost a wave per SIMD and the
    // solve time stays the same, so FP64 loads them where they are used
    constexpr bool kPre = sizeof(T) == 4;
    T bx[kPre ? N : 1];
    T uz[kPre ? N : 1];
    if constexpr (kPre) {
        if (pc.act) {
#pragma unroll
            for (int i = 0; i < N; ++i) bx[i] = bb[static_cast<int64_t>((i * N + pc.pa) * N + pc.pb) << G.logB];
            pencil_load<N, VP>(uz, uin + zpencil_base<N>(G, c, pc), G.logB);
        }
    }
    T y[N];
    wave_sipg_cell<N, T, VP, false>(uin, G, tb, F, c, L, y);   // ends synced
    TI* slab = kInT ? reinterpret_cast<TI*>(L.t) : reinterpret_cast<TI*>(&L);
    if (pc.act)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            T bv;
            if constexpr (kPre) bv = bx[i];
            else bv = bb[static_cast<int64_t>((i * N + pc.pa) * N + pc.pb) << G.logB];
            slab[SL::at(i, pc.pa, pc.pb)] = static_cast<TI>(bv - y[i]);
        }
    wave_sync();
    double d[N];
    wave_block_inverse<N, TI>(pc, slab, stab, stab + TABM, G, d);
    double s = 0.0;
    if (pc.act) {
        const int64_t pb = zpencil_base<N>(G, c, pc);
        double uv[N];
        if constexpr (kPre) {
#pragma unroll
            for (int k = 0; k < N; ++k) uv[k] = static_cast<double>(uz[k]);
        } else {
            pencil_load<N, VP>(uv, uin + pb, G.logB);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) uv[k] = fma(omega, d[k], uv[k]);
        pencil_store<N, VP>(uout + pb, uv, G.logB);
        if constexpr (DOT) {
            double rv[N];
            pencil_load<N, VP>(rv, r + pb, G.logB);
#pragma unroll
            for (int k = 0; k < N; ++k) s = fma(rv[k], static_cast<double>(static_cast<T>(uv[k])), s);
        }
    }
    if constexpr (DOT) {
        s = wave_sum(s);
        if (threadIdx.x == 0) part[c] = s;
    }
}

// (X (x) Y (x) Z) applied to the slab's block, in place, X acting on x:
// the lane's z-pencil z enters in registers; on return the lane holds its
// x-pencil (x0..x_{n-1} at (pa, pb) = (j, k)) of the result in out.
template <int N>
__device__ __forceinline__ void wave_kron3(const Pencil<N>& pc, double* slab, const double* X, const double* Y,
                                           const double* Z, const double (&z)[N], double (&out)[N]) {
    using SL = Slab<N>;
    if (pc.act) {   // z: lane (i, j)
#pragma unroll
        for (int k = 0; k < N; ++k) {
            double sacc = 0.0;
#pragma unroll
            for (int kk = 0; kk < N; ++kk) sacc = fma(Z[k * N + kk], z[kk], sacc);
            slab[SL::at(pc.pa, pc.pb, k)] = sacc;
        }
    }
    wave_sync();
    if (pc.act) {   // y: lane (i, k)
        double v[N];
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] = slab[SL::at(pc.pa, j, pc.pb)];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            double sacc = 0.0;
#pragma unroll
            for (int jj = 0; jj < N; ++jj) sacc = fma(Y[j * N + jj], v[jj], sacc);
            slab[SL::at(pc.pa, j, pc.pb)] = sacc;
        }
    }
    wave_sync();
    if (pc.act) {   // x: lane (j, k)
        double v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = slab[SL::at(i, pc.pa, pc.pb)];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            double sacc = 0.0;
#pragma unroll
            for (int ii = 0; ii < N; ++ii) sacc = fma(X[i * N + ii], v[ii], sacc);
            out[i] = sacc;
        }
    }
    wave_sync();
}

// b_coarse = P^T (b - A u), one coarse cell per workgroup of eight waves, one
// child per wave: the child's operator row by x-pencils, its residual turned
// to z-pencils in the wave's (by then free) operator scratch, the embedding's
// transpose, and the children's contributions summed in LDS in a fixed order.
// It is bound as the operator row is (vector instructions and LDS); the product
// and the residual no longer go through memory, and a level takes one launch
// less.  n = 8 in FP32: product and restriction 22 + 20 us on 24^3 cells, 8 + 6
// us on 12^3, against 35.5 and 9.9 us in one.
template <int N, bool VP, typename T = double>
__global__ __launch_bounds__(512, 2) void k_mg_coarsen_wave(const T* __restrict__ b, const T* __restrict__ u,
                                                            T* __restrict__ bc, MeshArgs G, MeshArgs Gc,
                                                            const T* __restrict__ tab, WaveFace<N, T> F,
                                                            ProlTab<N> PT, const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    using SL = Slab<N>;
    constexpr int N3 = N * N * N;
    constexpr int TAB = 2 * (EOShape<N>::SE + EOShape<N>::SO);
    static_assert(sizeof(WaveLds<N, T>) >= SL::size * sizeof(double) && sizeof(WaveLds<N, T>) % sizeof(double) == 0,
                  "residual slab in the operator scratch");
    __shared__ __align__(16) WaveLds<N, T> L[8];
    __shared__ double tabs[2 * N * N];
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.y);
    for (int e = ch * 64 + threadIdx.x; e < 2 * N * N; e += 512) tabs[e] = PT.p[e / (N * N)][e % (N * N)];
    T regs[sizeof(T) == 8 ? 1 : TAB];
    const T* tb = wave_row_tables<T, TAB>(regs, tab);
    const int64_t c = wave_tile(blockIdx.x, gridDim.x, Gc);
    const uint32_t cu = static_cast<uint32_t>(c);
    const uint32_t cz = cu % static_cast<uint32_t>(Gc.mz);
    const uint32_t rr = cu / static_cast<uint32_t>(Gc.mz);
    const uint32_t cy = rr % static_cast<uint32_t>(Gc.my);
    const uint32_t cx = rr / static_cast<uint32_t>(Gc.my);
    const int bx = ch >> 2, by = (ch >> 1) & 1, bz = ch & 1;
    const int64_t f = (static_cast<int64_t>(2 * cx + bx) * G.my + (2 * cy + by)) * G.mz + (2 * cz + bz);
    T y[N];
    wave_sipg_cell<N, T, VP, false>(u, G, tb, F, f, L[ch], y);   // ends synced
    const Pencil<N> pc(1);
    double* slab = reinterpret_cast<double*>(&L[ch]);
    if (pc.act) {
        const T* bb = b + G.offset + block_base(f, G.logB, N3);
#pragma unroll
        for (int i = 0; i < N; ++i)
            slab[SL::at(i, pc.pa, pc.pb)] =
                static_cast<double>(bb[static_cast<int64_t>((i * N + pc.pa) * N + pc.pb) << G.logB]) -
                static_cast<double>(y[i]);
    }
    tile_sync();
    double z[N], out[N];
    if (pc.act) {
#pragma unroll
        for (int k = 0; k < N; ++k) z[k] = slab[SL::at(pc.pa, pc.pb, k)];
    }
    wave_kron3<N>(pc, slab, tabs + bx * N * N, tabs + by * N * N, tabs + bz * N * N, z, out);
    if (pc.act) {
#pragma unroll
        for (int i = 0; i < N; ++i) slab[(i * N + pc.pa) * N + pc.pb] = out[i];
    }
    tile_sync();
    T* cb = bc + Gc.offset + block_base(c, Gc.logB, N3);
    for (int q = ch * 64 + threadIdx.x; q < N3; q += 512) {
        double s = reinterpret_cast<const double*>(&L[0])[q];
#pragma unroll
        for (int k = 1; k < 8; ++k) s += reinterpret_cast<const double*>(&L[k])[q];
        cb[static_cast<int64_t>(q) << Gc.logB] = static_cast<T>(s);
    }
}

// u_out = u_fine + P u_coarse, one fine cell per wave.
template <int N, bool VP, typename TS = double>
__global__ __launch_bounds__(64, 2) void k_mg_prolong_wave(const TS* __restrict__ uc,
                                                         const TS* __restrict__ uf, TS* __restrict__ uout,
                                                         MeshArgs Gf, MeshArgs Gc, ProlTab<N> P,
                                                         const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    __shared__ double slab[Slab<N>::size];
    __shared__ double tabs[2 * N * N];
    for (int e = threadIdx.x; e < 2 * N * N; e += 64) tabs[e] = P.p[e / (N * N)][e % (N * N)];
    wave_sync();
    const int64_t f = blockIdx.x;
    const uint32_t fu = static_cast<uint32_t>(f);
    const uint32_t fz = fu % static_cast<uint32_t>(Gf.mz);
    const uint32_t rr = fu / static_cast<uint32_t>(Gf.mz);
    const uint32_t fy = rr % static_cast<uint32_t>(Gf.my);
    const uint32_t fx = rr / static_cast<uint32_t>(Gf.my);
    const int64_t c = (static_cast<int64_t>(fx / 2) * Gc.my + fy / 2) * Gc.mz + fz / 2;
    const Pencil<N> pc(1);
    double z[N], out[N];
    if (pc.act) pencil_load<N, VP>(z, uc + zpencil_base<N>(Gc, c, pc), Gc.logB);
    wave_kron3<N>(pc, slab, tabs + (fx & 1) * N * N, tabs + (fy & 1) * N * N, tabs + (fz & 1) * N * N, z, out);
    if (pc.act) {
        const int64_t base = Gf.offset + block_base(f, Gf.logB, N * N * N);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int64_t o = base + (static_cast<int64_t>((i * N + pc.pa) * N + pc.pb) << Gf.logB);
            uout[o] = static_cast<TS>(static_cast<double>(uf[o]) + out[i]);
        }
    }
}

// Partial (a, b) per cell, one cell per wave.
template <int N, bool VP, typename TB = double>
__global__ __launch_bounds__(64) void k_mg_dot_wave(const double* __restrict__ a, const TB* __restrict__ b,
                                                    MeshArgs G, double* __restrict__ part,
                                                    const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    const int64_t c = blockIdx.x;
    const Pencil<N> pc(1);
    double s = 0.0;
    if (pc.act) {
        const int64_t pb = zpencil_base<N>(G, c, pc);
        double av[N], bv[N];
        pencil_load<N, VP>(av, a + pb, G.logB);
        pencil_load<N, VP>(bv, b + pb, G.logB);
#pragma unroll
        for (int k = 0; k < N; ++k) s = fma(av[k], bv[k], s);
    }
    s = wave_sum(s);
    if (threadIdx.x == 0) part[c] = s;
}

// The degree-coarsened coarsest level (n >= 5, Lagrange basis), used when
// the coarsest geometric level is too large for the dense solve: on the
// same cells the degree drops to 1 (eight unknowns per cell in canonical
// order, contiguous per cell), reached by the cellwise embedding
// E = E1 (x) E1 (x) E1 of Q_1 into Q_p, E1[i] = (1 - x_i, x_i) at the nodes
// x_i of [0, 1]; its operator is the Galerkin product E^T A E.
template <int N>
struct DegTab {
    double e[N][2];
};

// bc = E^T (b - t), one cell per wave: lane (a, q) sums its z-pencil against
// both coarse z functions, the eight coarse unknowns are wave sums.
template <int N, typename TS = double>
__global__ __launch_bounds__(64) void k_mg_deg_restrict(const TS* __restrict__ b, const TS* __restrict__ t,
                                                        double* __restrict__ bc, MeshArgs G, DegTab<N> E,
                                                        const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    const int64_t c = blockIdx.x;
    const Pencil<N> pc(1);
    double s0 = 0.0, s1 = 0.0, ex[2] = {0.0, 0.0}, ey[2] = {0.0, 0.0};
    if (pc.act) {
        const int64_t pb = zpencil_base<N>(G, c, pc);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int64_t o = pb + (static_cast<int64_t>(k) << G.logB);
            const double v = static_cast<double>(b[o]) - static_cast<double>(t[o]);
            s0 = fma(E.e[k][0], v, s0);
            s1 = fma(E.e[k][1], v, s1);
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                ex[j] = pc.pa == i ? E.e[i][j] : ex[j];
                ey[j] = pc.pb == i ? E.e[i][j] : ey[j];
            }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const double v = wave_sum(ex[j >> 2] * ey[(j >> 1) & 1] * ((j & 1) ? s1 : s0));
        if (threadIdx.x == 0) bc[c * 8 + j] = v;
    }
}

// uout = u + E uc, one thread per fine unknown.
template <int N, typename TS = double>
__global__ __launch_bounds__(64) void k_mg_deg_prolong(const double* __restrict__ uc, const TS* __restrict__ u,
                                                       TS* __restrict__ uout, MeshArgs G, DegTab<N> E,
                                                       const PcgState* __restrict__ st) {
    if (done_flag(st)) return;
    constexpr int N3 = N * N * N;
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x;
    if (idx >= G.ncells * N3) return;
    const int64_t c = idx / N3;
    const int q = static_cast<int>(idx % N3);
    const int a = q / (N * N), y = (q / N) % N, k = q % N;
    const double* v = uc + c * 8;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) s = fma(E.e[a][j >> 2] * E.e[y][(j >> 1) & 1] * E.e[k][j & 1], v[j], s);
    const int64_t o = G.offset + block_base(c, G.logB, N3) + (static_cast<int64_t>(q) << G.logB);
    uout[o] = static_cast<TS>(static_cast<double>(u[o]) + s);
}

template <int N>
DegTab<N> deg_table() {
    DegTab<N> E;
    double x[N];
    gll_points(N, x);
    for (int i = 0; i < N; ++i) E.e[i][0] = 1.0 - x[i], E.e[i][1] = x[i];
    return E;
}

// dst = src converted element by element (the finest level's right-hand
// side into the FP32-storage hierarchy, its result back to FP64).  Elements
// [full, n) are a ragged last tile, of which the `rest` first lanes of mask + 1
// hold cells: the caller's padding lanes are not written.
template <typename TD, typename TSRC>
__global__ __launch_bounds__(256) void k_mg_convert(const TSRC* __restrict__ src, TD* __restrict__ dst, int64_t n,
                                                    int64_t full, int mask, int rest) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * 256)
        if (i < full || (static_cast<int>(i) & mask) < rest) dst[i] = static_cast<TD>(src[i]);
}

tp_status check_launch(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, what);
    return TP_OK;
}

// Cholesky factorization and inverse of a symmetric positive definite
// matrix (row-major), the triangular solves spread over host threads;
// the inverse is returned column-major (equal to row-major: symmetric).
bool spd_inverse(int64_t n, std::vector<double>& A, std::vector<double>& inv) {
    for (int64_t j = 0; j < n; ++j) {
        double d = A[j * n + j];
        for (int64_t k = 0; k < j; ++k) d -= A[j * n + k] * A[j * n + k];
        if (!(d > 0.0)) return false;
        const double l = std::sqrt(d);
        A[j * n + j] = l;
        for (int64_t i = j + 1; i < n; ++i) {
            double s = A[i * n + j];
            for (int64_t k = 0; k < j; ++k) s -= A[i * n + k] * A[j * n + k];
            A[i * n + j] = s / l;
        }
    }
    inv.assign(static_cast<size_t>(n * n), 0.0);
    const unsigned nt = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    auto work = [&](unsigned tid) {
        std::vector<double> y(static_cast<size_t>(n));
        for (int64_t col = tid; col < n; col += nt) {
            for (int64_t i = 0; i < n; ++i) {       // L y = e_col
                double s = i == col ? 1.0 : 0.0;
                for (int64_t k = 0; k < i; ++k) s -= A[i * n + k] * y[k];
                y[i] = s / A[i * n + i];
            }
            for (int64_t i = n - 1; i >= 0; --i) {  // L^T x = y
                double s = y[i];
                for (int64_t k = i + 1; k < n; ++k) s -= A[k * n + i] * inv[col * n + k];
                inv[col * n + i] = s / A[i * n + i];
            }
        }
    };
    std::vector<std::thread> th;
    for (unsigned t = 0; t < nt; ++t) th.emplace_back(work, t);
    for (auto& t : th) t.join();
    return true;
}

}  // namespace

// Coarse inverses are shared by every hierarchy with the same coarsest level
// on a device and kept until the process ends.
struct CoarseKey {
    int device, n, basis, deg, mx, my, mz;
    double hx, hy, hz, C;
    bool operator<(const CoarseKey& o) const {
        return std::tie(device, n, basis, deg, mx, my, mz, hx, hy, hz, C) <
               std::tie(o.device, o.n, o.basis, o.deg, o.mx, o.my, o.mz, o.hx, o.hy, o.hz, o.C);
    }
};
static std::mutex g_coarse_mutex;
static std::map<CoarseKey, double*> g_coarse;

}  // namespace tpfdm

using namespace tpfdm;

struct MgLevel {
    MeshArgs G;
    int64_t elems = 0;
    void* t = nullptr;     // residual scratch
    void* b = nullptr;     // right-hand side (levels below the finest; every level with FP32 storage)
    void* u = nullptr;     // correction (levels below the finest; every level with FP32 storage)
};

struct tp_mg {
    tp_plan* plan = nullptr;
    int n = 0;
    int storage = TP_F64;           // element type of the level vectors (TP_F64 or TP_F32)
    std::vector<MgLevel> lv;
    double omega[3] = {0.0, 0.0, 0.0};
    double* coarse_inv = nullptr;   // shared, not owned
    int64_t n0 = 0;
    // degree-coarsened coarsest level (n >= 5): degree 1 on the last
    // geometric level's cells, right-hand side and correction of n0 values
    bool deg = false;
    double* deg_b = nullptr;
    double* deg_u = nullptr;
};

namespace {

// Where the finest level's last update leaves the partials of (r, u): count of
// them in part (0: it did not, as when the finest level has no update of its
// own).  r in FP64, 16-byte aligned.
struct RzPartials {
    const double* r;
    double* part;
    int64_t count;
};

// Embeddings into the children and their transposes.
template <int N>
void prolongation_tables(const Plan& plan, ProlTab<N>& P, ProlTab<N>& PT) {
    for (int i = 0; i < N * N; ++i) P.p[0][i] = plan.ref[N].P0[i], P.p[1][i] = plan.ref[N].P1[i];
    for (int c = 0; c < 2; ++c)
        for (int i = 0; i < N; ++i)
            for (int j = 0; j < N; ++j) PT.p[c][i * N + j] = P.p[c][j * N + i];
}

template <int N, typename TI, bool HERM, typename TS>
tp_status vcycle_level(const tp_mg* m, size_t l, const TS* b, TS* u, const PcgState* st, hipStream_t s,
                       RzPartials* rz = nullptr) {
    const Plan& plan = *m->plan;
    const MgLevel& L = m->lv[l];
    TS* Lt = static_cast<TS*>(L.t);
    const unsigned grid = static_cast<unsigned>((L.G.ncells + 63) / 64);
    if (l + 1 == m->lv.size()) {
        hipLaunchKernelGGL((k_mg_coarse<N, TS>), dim3(coarse_grid(m->n0)), dim3(64, kCoarseRows), 0, s, m->coarse_inv,
                           b, u, static_cast<int>(m->n0), L.G.offset, L.G.logB, st);
        return check_launch("coarse solve");
    }
    const TileTab<N, MgTC<TS>, HERM> R = tile_tab<N, MgTC<TS>, HERM>(plan, false);
    if (L.G.ncells <= 64 && m->n0 <= kTailUnknowns) {   // (at most three levels: 64, 8 and 1 cells)
        TailArgs<N, TI, HERM, TS> M;
        M.levels = static_cast<int>(m->lv.size() - l);
        M.n0 = static_cast<int>(m->n0);
        M.R = R;
        for (int i = 0; i < M.levels; ++i) {
            M.G[i] = m->lv[l + i].G;
            if (i + 1 < M.levels) M.E[i] = tile_inv<N, TI>(plan.ref[N], M.G[i]);
        }
        prolongation_tables<N>(plan, M.P, M.PT);
        for (int j = 0; j < 3; ++j) M.omega[j] = m->omega[j];
        M.inv = m->coarse_inv;
        hipLaunchKernelGGL((k_mg_tail<N, TI, HERM, TS>), dim3(1), dim3(64, N), 0, s, b, u, M, st);
        return check_launch("coarse levels");
    }
    const TileInv<N, TI> E = tile_inv<N, TI>(plan.ref[N], L.G);
    ProlTab<N> P, PT;
    prolongation_tables<N>(plan, P, PT);
    const bool pairs = tile_pairs(L.G, sizeof(TS), reinterpret_cast<uintptr_t>(b) % 16 == 0 &&
                                                       reinterpret_cast<uintptr_t>(u) % 16 == 0);
    // Chebyshev updates ping-pong between u and the level's scratch t; the
    // prolongation writes out of place so that the last update lands in u.
    auto step = [&](const TS* from, TS* to, int j) {
        if constexpr (sizeof(TS) == 8) {
            if (pairs) {
                hipLaunchKernelGGL((k_mg_smooth<N, TI, HERM, TS, 2>), dim3(tile_grid(L.G, 2)), dim3(64, N), 0, s, b,
                                   from, to, L.G, R, E, m->omega[j], st, nullptr, nullptr);
                return;
            }
        }
        hipLaunchKernelGGL((k_mg_smooth<N, TI, HERM, TS>), dim3(grid), dim3(64, N), 0, s, b, from, to, L.G, R, E,
                           m->omega[j], st, nullptr, nullptr);
    };
    // the last update, with the partials of (r, u) when they are asked for
    auto last_step = [&](const TS* from, TS* to, int j) {
        if (!rz) return step(from, to, j);
        if constexpr (sizeof(TS) == 8) {
            if (pairs) {
                rz->count = tile_grid(L.G, 2);
                hipLaunchKernelGGL((k_mg_smooth<N, TI, HERM, TS, 2, true>), dim3(tile_grid(L.G, 2)), dim3(64, N), 0, s,
                                   b, from, to, L.G, R, E, m->omega[j], st, rz->r, rz->part);
                return;
            }
        }
        rz->count = grid;
        hipLaunchKernelGGL((k_mg_smooth<N, TI, HERM, TS, 1, true>), dim3(grid), dim3(64, N), 0, s, b, from, to, L.G, R,
                           E, m->omega[j], st, rz->r, rz->part);
    };
    hipLaunchKernelGGL((k_mg_jacobi0<N, TI, TS>), dim3(grid), dim3(64, N), 0, s, b, u, L.G, E,
                       m->omega[0], st);
    step(u, Lt, 1);
    step(Lt, u, 2);
    const MgLevel& C = m->lv[l + 1];
    TS* Cb = static_cast<TS*>(C.b);
    TS* Cu = static_cast<TS*>(C.u);
    bool wide = false;
    if constexpr (sizeof(TS) == 8) {
        wide = pairs;
        if (wide)
            hipLaunchKernelGGL((k_mg_apply<N, HERM, TS, 2>), dim3(tile_grid(L.G, 2)), dim3(64, N), 0, s, u, Lt, L.G,
                               R, st);
    }
    if (!wide)
        hipLaunchKernelGGL((k_mg_apply<N, HERM, TS>), dim3(grid), dim3(64, N), 0, s, u, Lt, L.G, R, st);
    hipLaunchKernelGGL((k_mg_restrict<N, TS>), dim3(tile_grid(C.G, 1)), dim3(64, 2 * N), 0, s, b, Lt, Cb, L.G, C.G,
                       PT, st);
    tp_status stt = check_launch("level transfer");
    if (stt != TP_OK) return stt;
    stt = vcycle_level<N, TI, HERM, TS>(m, l + 1, Cb, Cu, st, s);
    if (stt != TP_OK) return stt;
    hipLaunchKernelGGL((k_mg_prolong<N, TS>), dim3(grid), dim3(64, N), 0, s, Cu, u, Lt, L.G, C.G, P, st);
    step(Lt, u, 0);
    step(u, Lt, 1);
    last_step(Lt, u, 2);
    return check_launch("smoothing");
}

// The same V-cycle for n >= 5 on the wave kernels (layout B = 1: pencils
// move as 16-byte vectors where VP), level vectors and operator rows in TS
// (FP64, or FP32 for the FP32-storage hierarchy).
template <int N, typename TI, bool VP, typename TS>
tp_status vcycle_level_wave(const tp_mg* m, size_t l, const TS* b, TS* u, const PcgState* st, hipStream_t s,
                            RzPartials* rz = nullptr) {
    const Plan& plan = *m->plan;
    const MgLevel& L = m->lv[l];
    TS* Lt = static_cast<TS*>(L.t);
    const unsigned grid = static_cast<unsigned>(L.G.ncells);
    const bool last = l + 1 == m->lv.size();
    if (last && !m->deg) {
        hipLaunchKernelGGL((k_mg_coarse<N, TS>), dim3(coarse_grid(m->n0)), dim3(64, kCoarseRows), 0, s, m->coarse_inv,
                           b, u, static_cast<int>(m->n0), L.G.offset, L.G.logB, st);
        return check_launch("coarse solve");
    }
    const WaveFace<N, TS> F = wave_face<N, TS>(plan);
    const TS* tabA = reinterpret_cast<const TS*>(eo_table(plan, N, EO_APPLY_A, sizeof(TS) == 8 ? 0 : 1));
    const TI* tabS = reinterpret_cast<const TI*>(eo_table(plan, N, EO_INV, sizeof(TI) == 8 ? 0 : 1));
    ProlTab<N> P, PT;
    prolongation_tables<N>(plan, P, PT);
    auto step = [&](const TS* from, TS* to, int j) {
        hipLaunchKernelGGL((k_mg_smooth_wave<N, TI, VP, TS>), dim3(grid), dim3(64), 0, s, b, from, to, L.G, tabA, F,
                           tabS, m->omega[j], st, nullptr, nullptr);
    };
    // the last update, with the partials of (r, u) when they are asked for
    auto last_step = [&](const TS* from, TS* to, int j) {
        if (!rz) return step(from, to, j);
        rz->count = grid;
        hipLaunchKernelGGL((k_mg_smooth_wave<N, TI, VP, TS, true>), dim3(grid), dim3(64), 0, s, b, from, to, L.G, tabA,
                           F, tabS, m->omega[j], st, rz->r, rz->part);
    };
    hipLaunchKernelGGL((k_mg_jacobi0_wave<N, TI, VP, TS>), dim3(grid), dim3(64), 0, s, b, u, L.G, tabS, m->omega[0],
                       st);
    step(u, Lt, 1);
    step(Lt, u, 2);
    if (last) {
        // coarse correction on the degree-1 level: E^T (b - A u), its dense
        // solve, u + E u_c
        const DegTab<N> E = deg_table<N>();
        hipLaunchKernelGGL((k_mg_apply_wave<N, VP, TS>), dim3(grid), dim3(64), 0, s, u, Lt, L.G, tabA, F, st);
        hipLaunchKernelGGL((k_mg_deg_restrict<N, TS>), dim3(grid), dim3(64), 0, s, b, Lt, m->deg_b, L.G, E, st);
        hipLaunchKernelGGL((k_mg_coarse<2, double>), dim3(coarse_grid(m->n0)), dim3(64, kCoarseRows), 0, s,
                           m->coarse_inv, m->deg_b, m->deg_u, static_cast<int>(m->n0), int64_t(0), 0, st);
        hipLaunchKernelGGL((k_mg_deg_prolong<N, TS>),
                           dim3(static_cast<unsigned>((L.G.ncells * N * N * N + 63) / 64)), dim3(64), 0, s, m->deg_u,
                           u, Lt, L.G, E, st);
        tp_status stt = check_launch("degree-level correction");
        if (stt != TP_OK) return stt;
        step(Lt, u, 0);
        step(u, Lt, 1);
        last_step(Lt, u, 2);
        return check_launch("smoothing");
    }
    const MgLevel& C = m->lv[l + 1];
    TS* Cb = static_cast<TS*>(C.b);
    TS* Cu = static_cast<TS*>(C.u);
    hipLaunchKernelGGL((k_mg_coarsen_wave<N, VP, TS>), dim3(static_cast<unsigned>(C.G.ncells)), dim3(64, 8), 0, s, b, u,
                       Cb, L.G, C.G, tabA, F, PT, st);
    tp_status stt = check_launch("level transfer");
    if (stt != TP_OK) return stt;
    stt = vcycle_level_wave<N, TI, VP, TS>(m, l + 1, Cb, Cu, st, s);
    if (stt != TP_OK) return stt;
    hipLaunchKernelGGL((k_mg_prolong_wave<N, VP, TS>), dim3(grid), dim3(64), 0, s, Cu, u, Lt, L.G, C.G, P, st);
    step(Lt, u, 0);
    step(u, Lt, 1);
    last_step(Lt, u, 2);
    return check_launch("smoothing");
}

template <typename TI, typename TS>
tp_status vcycle_dispatch(const tp_mg* m, const TS* b, TS* u, const PcgState* st, hipStream_t s,
                          RzPartials* rz) {
    switch (m->n) {
        case 2: return vcycle_level<2, TI, false, TS>(m, 0, b, u, st, s, rz);
        case 3: return vcycle_level<3, TI, false, TS>(m, 0, b, u, st, s, rz);
        case 4:
            return m->plan->basis == TP_BASIS_HERMITE ? vcycle_level<4, TI, true, TS>(m, 0, b, u, st, s, rz)
                                                      : vcycle_level<4, TI, false, TS>(m, 0, b, u, st, s, rz);
        default: break;
    }
    {
        // 16-byte pencil accesses when the caller's finest b and u allow them
        // (the level vectors are allocation-aligned) and a pencil is a whole
        // number of 16-byte vectors
        const bool vp = reinterpret_cast<uintptr_t>(b) % 16 == 0 && reinterpret_cast<uintptr_t>(u) % 16 == 0;
        constexpr bool v6 = (6 * sizeof(TS)) % 16 == 0;
        switch (m->n) {
            case 5: return vcycle_level_wave<5, TI, false, TS>(m, 0, b, u, st, s, rz);
            case 6: return vp && v6 ? vcycle_level_wave<6, TI, v6, TS>(m, 0, b, u, st, s, rz)
                                    : vcycle_level_wave<6, TI, false, TS>(m, 0, b, u, st, s, rz);
            case 7: return vcycle_level_wave<7, TI, false, TS>(m, 0, b, u, st, s, rz);
            case 8: return vp ? vcycle_level_wave<8, TI, true, TS>(m, 0, b, u, st, s, rz)
                              : vcycle_level_wave<8, TI, false, TS>(m, 0, b, u, st, s, rz);
            default: break;
        }
    }
    return set_error(TP_ERR_UNSUPPORTED, "multigrid supports n <= 8");
}

template <int N>
tp_status coarse_probe_n(const tp_mg* m, std::vector<double>& A) {
    const Plan& plan = *m->plan;
    const MgLevel& L = m->lv.back();
    const WaveFace<N, double> F = wave_face<N, double>(plan);
    constexpr int N3 = N * N * N;
    const int64_t n0 = m->n0;
    A.assign(static_cast<size_t>(n0 * n0), 0.0);
    std::vector<double> col(static_cast<size_t>(L.elems));
    const unsigned grid = static_cast<unsigned>((L.G.ncells + 63) / 64);
    // FP64 probe vectors of the coarsest level (freed on return)
    double *pu = nullptr, *pt = nullptr;
    const size_t vb = static_cast<size_t>(L.elems) * sizeof(double);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&pu), vb);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&pt), vb);
    tp_status st = e == hipSuccess ? TP_OK : hip_error(e, "coarse probe vectors");
    bool herm = false;
    // column j = A e_j, with pu = e_j as the probe
    for (int64_t j = 0; st == TP_OK && j < n0; ++j) {
        st = launch_fill(pu, L.elems, TP_F64, 0, true, nullptr);
        if (st != TP_OK) break;
        const double one = 1.0;
        const int64_t pos = L.G.offset + block_base(j / N3, L.G.logB, N3) + ((j % N3) << L.G.logB);
        e = hipMemcpy(pu + pos, &one, sizeof(double), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            st = hip_error(e, "coarse probe");
            break;
        }
        if constexpr (N <= kLaneMaxN) {
            const PcgState* none = nullptr;
            if constexpr (N == 4) {
                if (plan.basis == TP_BASIS_HERMITE) {
                    hipLaunchKernelGGL((k_mg_apply<N, true, double>), dim3(grid), dim3(64, N), 0, nullptr, pu, pt, L.G,
                                       tile_tab<N, double, true>(plan, false), none);
                    herm = true;
                }
            }
            if (!herm)
                hipLaunchKernelGGL((k_mg_apply<N, false, double>), dim3(grid), dim3(64, N), 0, nullptr, pu, pt, L.G,
                                   tile_tab<N, double, false>(plan, false), none);
        }
        else
            hipLaunchKernelGGL((k_mg_apply_wave<N, false>), dim3(static_cast<unsigned>(L.G.ncells)), dim3(64), 0,
                               nullptr, pu, pt, L.G, reinterpret_cast<const double*>(eo_table(plan, N, EO_APPLY_A, 0)),
                               F, static_cast<const PcgState*>(nullptr));
        e = hipMemcpy(col.data(), pt, vb, hipMemcpyDeviceToHost);
        if (e != hipSuccess) {
            st = hip_error(e, "coarse probe");
            break;
        }
        for (int64_t i = 0; i < n0; ++i)
            A[i * n0 + j] =
                col[static_cast<size_t>(L.G.offset + block_base(i / N3, L.G.logB, N3) + ((i % N3) << L.G.logB))];
    }
    if (pu) (void)hipFree(pu);
    if (pt) (void)hipFree(pt);
    return st;
}

// The Galerkin operator E^T A E of the degree-1 level, column by column:
// E e_j on the last geometric level, A of it, then E^T of that.
template <int N>
tp_status coarse_probe_deg(const tp_mg* m, std::vector<double>& A) {
    const Plan& plan = *m->plan;
    const MgLevel& L = m->lv.back();
    const WaveFace<N, double> F = wave_face<N, double>(plan);
    const double* tabA = reinterpret_cast<const double*>(eo_table(plan, N, EO_APPLY_A, 0));
    const DegTab<N> E = deg_table<N>();
    const int64_t n0 = m->n0;
    A.assign(static_cast<size_t>(n0 * n0), 0.0);
    std::vector<double> col(static_cast<size_t>(n0));
    // FP64 probe vectors (freed on return): zero, E e_j and A E e_j on the
    // last geometric level, e_j and the column on the degree-1 level
    double *zf = nullptr, *pu = nullptr, *pt = nullptr, *ec = nullptr, *cc = nullptr;
    const size_t vb = static_cast<size_t>(L.elems) * sizeof(double);
    const size_t cb = static_cast<size_t>(n0) * sizeof(double);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&zf), vb);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&pu), vb);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&pt), vb);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&ec), cb);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&cc), cb);
    tp_status st = e == hipSuccess ? TP_OK : hip_error(e, "degree-level probe vectors");
    if (st == TP_OK) st = launch_fill(zf, L.elems, TP_F64, 0, true, nullptr);
    if (st == TP_OK) st = launch_fill(pu, L.elems, TP_F64, 0, true, nullptr);
    const PcgState* none = nullptr;
    const unsigned gf = static_cast<unsigned>((L.G.ncells * N * N * N + 63) / 64);
    for (int64_t j = 0; st == TP_OK && j < n0; ++j) {
        st = launch_fill(ec, n0, TP_F64, 0, true, nullptr);
        if (st != TP_OK) break;
        const double one = 1.0;
        e = hipMemcpy(ec + j, &one, sizeof(double), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            st = hip_error(e, "degree-level probe");
            break;
        }
        hipLaunchKernelGGL((k_mg_deg_prolong<N>), dim3(gf), dim3(64), 0, nullptr, ec, zf, pu, L.G, E, none);
        hipLaunchKernelGGL((k_mg_apply_wave<N, false>), dim3(static_cast<unsigned>(L.G.ncells)), dim3(64), 0, nullptr,
                           pu, pt, L.G, tabA, F, none);
        hipLaunchKernelGGL((k_mg_deg_restrict<N>), dim3(static_cast<unsigned>(L.G.ncells)), dim3(64), 0, nullptr, pt, zf,
                           cc, L.G, E, none);
        st = check_launch("degree-level probe");
        if (st != TP_OK) break;
        e = hipMemcpy(col.data(), cc, cb, hipMemcpyDeviceToHost);
        if (e != hipSuccess) {
            st = hip_error(e, "degree-level probe");
            break;
        }
        for (int64_t i = 0; i < n0; ++i) A[i * n0 + j] = col[static_cast<size_t>(i)];
    }
    for (double* q : {zf, pu, pt, ec, cc})
        if (q) (void)hipFree(q);
    return st;
}

void free_mg(tp_mg* m) {
    for (auto& L : m->lv)
        for (void* p : {L.t, L.b, L.u})
            if (p) (void)hipFree(p);
    m->lv.clear();
    for (double* p : {m->deg_b, m->deg_u})
        if (p) (void)hipFree(p);
    m->deg_b = m->deg_u = nullptr;
}

template <int N, bool VP>
void launch_dot_wave(const MgLevel& L, const double* a, const void* b, bool b32, double* part, const PcgState* ps,
                     hipStream_t s) {
    const unsigned grid = static_cast<unsigned>(L.G.ncells);
    if (b32)
        hipLaunchKernelGGL((k_mg_dot_wave<N, VP, float>), dim3(grid), dim3(64), 0, s, a, static_cast<const float*>(b),
                           L.G, part, ps);
    else
        hipLaunchKernelGGL((k_mg_dot_wave<N, VP, double>), dim3(grid), dim3(64), 0, s, a, static_cast<const double*>(b),
                           L.G, part, ps);
}

tp_status convert_launch(const void* src, void* dst, bool to_f32, const tp_mg* m, hipStream_t s) {
    const MgLevel& L = m->lv[0];
    const int64_t n = L.elems, n3 = int64_t(m->n) * m->n * m->n;
    const int64_t full = (L.G.ncells >> L.G.logB) * n3 << L.G.logB;
    const int mask = (1 << L.G.logB) - 1, rest = static_cast<int>(L.G.ncells) & mask;
    const unsigned grid = static_cast<unsigned>(std::min<int64_t>((n + 255) / 256, 8192));
    if (to_f32)
        hipLaunchKernelGGL((k_mg_convert<float, double>), dim3(grid), dim3(256), 0, s, static_cast<const double*>(src),
                           static_cast<float*>(dst), n, full, mask, rest);
    else
        hipLaunchKernelGGL((k_mg_convert<double, float>), dim3(grid), dim3(256), 0, s, static_cast<const float*>(src),
                           static_cast<double*>(dst), n, full, mask, rest);
    return check_launch("multigrid conversion");
}

}  // namespace

namespace tpfdm {
namespace {
// The cycle on the finest level's vectors: with FP32 level storage its own
// right-hand side and result.
tp_status vcycle_on_level(const tp_mg* m, const double* b, double* u, const PcgState* ps, bool f32, hipStream_t s,
                          RzPartials* rz) {
    // the smoother reads the plan's cell-block eigen tables at every enqueue
    if (m->plan->inverse_op != TP_OP_CELL || m->plan->factor_mode != TP_FACTOR_SCALED)
        return set_error(TP_ERR_STATE, "the plan's inverse setup is no longer TP_OP_CELL, TP_FACTOR_SCALED");
    if (m->storage == TP_F32) {
        const float* b32 = static_cast<const float*>(m->lv[0].b);
        float* u32 = static_cast<float*>(m->lv[0].u);
        return f32 ? vcycle_dispatch<float, float>(m, b32, u32, ps, s, rz)
                   : vcycle_dispatch<double, float>(m, b32, u32, ps, s, rz);
    }
    return f32 ? vcycle_dispatch<float, double>(m, b, u, ps, s, rz)
               : vcycle_dispatch<double, double>(m, b, u, ps, s, rz);
}
}  // namespace

tp_status mg_enqueue_vcycle(const tp_mg* m, const double* b, double* u, bool f32, hipStream_t s) {
    if (m->storage != TP_F32) return vcycle_on_level(m, b, u, nullptr, f32, s, nullptr);
    // b into the hierarchy's FP32 right-hand side, the cycle, and (when u is
    // given) the FP32 result back to FP64
    const MgLevel& L0 = m->lv[0];
    tp_status r = convert_launch(b, L0.b, true, m, s);
    if (r == TP_OK) r = vcycle_on_level(m, nullptr, nullptr, nullptr, f32, s, nullptr);
    if (r != TP_OK || !u) return r;
    return convert_launch(L0.u, u, false, m, s);
}

tp_status mg_enqueue_iteration(const tp_mg* m, const double* r, double* z, double* part, int64_t* count, const void* st,
                               bool f32, hipStream_t s) {
    const PcgState* ps = static_cast<const PcgState*>(st);
    const bool f32s = m->storage == TP_F32;
    RzPartials rz{r, part, 0};
    tp_status e = vcycle_on_level(m, r, z, ps, f32, s, &rz);
    if (e == TP_OK && rz.count == 0) {
        rz.count = m->n <= kLaneMaxN ? (m->lv[0].G.ncells + 63) / 64 : m->lv[0].G.ncells;
        e = mg_enqueue_dot(m, r, f32s ? m->lv[0].u : static_cast<const void*>(z), f32s, part, st, s);
    }
    *count = rz.count;
    return e;
}

float* mg_rhs32(const tp_mg* m) { return m->storage == TP_F32 ? static_cast<float*>(m->lv[0].b) : nullptr; }

int mg_storage(const tp_mg* m) { return m->storage; }

const float* mg_result32(const tp_mg* m) {
    return m->storage == TP_F32 ? static_cast<const float*>(m->lv[0].u) : nullptr;
}

tp_status mg_enqueue_dot(const tp_mg* m, const double* a, const void* b, bool b32, double* part, const void* st,
                         hipStream_t s) {
    const MgLevel& L = m->lv[0];
    // 16-byte pencil loads for n = 8 (and n = 6 with FP64 b) when both
    // vectors are 16-byte aligned (solver and level vectors are)
    const bool vp = reinterpret_cast<uintptr_t>(a) % 16 == 0 && reinterpret_cast<uintptr_t>(b) % 16 == 0;
    const unsigned grid = static_cast<unsigned>((L.G.ncells + 63) / 64);
    const PcgState* ps = static_cast<const PcgState*>(st);
    const double* bd = static_cast<const double*>(b);
    const float* bf = static_cast<const float*>(b);
    switch (m->n) {
        case 2:
            if (b32) hipLaunchKernelGGL((k_mg_dot<2, float>), dim3(grid), dim3(64), 0, s, a, bf, L.G, part, ps);
            else hipLaunchKernelGGL((k_mg_dot<2, double>), dim3(grid), dim3(64), 0, s, a, bd, L.G, part, ps);
            break;
        case 3:
            if (b32) hipLaunchKernelGGL((k_mg_dot<3, float>), dim3(grid), dim3(64), 0, s, a, bf, L.G, part, ps);
            else hipLaunchKernelGGL((k_mg_dot<3, double>), dim3(grid), dim3(64), 0, s, a, bd, L.G, part, ps);
            break;
        case 4:
            if (b32) hipLaunchKernelGGL((k_mg_dot<4, float>), dim3(grid), dim3(64), 0, s, a, bf, L.G, part, ps);
            else hipLaunchKernelGGL((k_mg_dot<4, double>), dim3(grid), dim3(64), 0, s, a, bd, L.G, part, ps);
            break;
        case 5: launch_dot_wave<5, false>(L, a, b, b32, part, ps, s); break;
        case 6:
            if (vp && !b32) launch_dot_wave<6, true>(L, a, b, b32, part, ps, s);
            else launch_dot_wave<6, false>(L, a, b, b32, part, ps, s);
            break;
        case 7: launch_dot_wave<7, false>(L, a, b, b32, part, ps, s); break;
        case 8:
            if (vp) launch_dot_wave<8, true>(L, a, b, b32, part, ps, s);
            else launch_dot_wave<8, false>(L, a, b, b32, part, ps, s);
            break;
        default: return set_error(TP_ERR_UNSUPPORTED, "multigrid supports n <= 8");
    }
    return check_launch("dot");
}

tp_status mg_enqueue_widen(const tp_mg* m, double* dst, hipStream_t s) {
    if (m->storage != TP_F32) return set_error(TP_ERR_STATE, "the multigrid stores its levels in FP64");
    return convert_launch(m->lv[0].u, dst, false, m, s);
}

const tp_plan* mg_plan(const tp_mg* m) { return m->plan; }
}  // namespace tpfdm

extern "C" {

tp_status tp_mg_create(tp_plan* plan, tp_mg** out) { return tp_mg_create_typed(plan, TP_F64, out); }

tp_status tp_mg_create_typed(tp_plan* plan, tp_dtype storage, tp_mg** out) {
    if (!out) return set_error(TP_ERR_ARG, "out must be non-null");
    *out = nullptr;
    if (!plan) return set_error(TP_ERR_ARG, "plan is null");
    if (storage != TP_F64 && storage != TP_F32)
        return set_error(TP_ERR_UNSUPPORTED, "multigrid level vectors are stored in FP64 or FP32");
    if (!plan->mesh) return set_error(TP_ERR_UNSUPPORTED, "multigrid needs a mesh plan");
    const GroupInfo& g = plan->groups[0];
    if (g.n <= kLaneMaxN && g.logB != 6)
        return set_error(TP_ERR_UNSUPPORTED, "multigrid needs the layout B = 64 for n <= 4");
    if (g.n > kLaneMaxN && g.logB != 0)
        return set_error(TP_ERR_UNSUPPORTED, "multigrid needs the layout B = 1 for n >= 5");
    if (g.n > kLaneMaxN && plan->basis == TP_BASIS_HERMITE)
        return set_error(TP_ERR_UNSUPPORTED, "multigrid in the Hermite-type basis supports n = 4");
    if (plan->inverse_op != TP_OP_CELL || plan->factor_mode != TP_FACTOR_SCALED)
        return set_error(TP_ERR_STATE, "multigrid needs tp_setup_inverse(TP_OP_CELL, TP_FACTOR_SCALED) first");
    tp_mg* m = new (std::nothrow) tp_mg();
    if (!m) return set_error(TP_ERR_OOM, "host allocation failed");
    m->plan = plan;
    m->n = g.n;
    m->storage = storage;
    const size_t es = storage == TP_F32 ? sizeof(float) : sizeof(double);
    const double a = 0.2, b = 2.0, c = 0.5 * (a + b), d = 0.5 * (b - a);
    for (int j = 1; j <= 3; ++j) m->omega[j - 1] = 1.0 / (c - d * std::cos((2 * j - 1) * 3.141592653589793 / 6.0));
    // levels
    int mx = plan->mesh_m[0], my = plan->mesh_m[1], mz = plan->mesh_m[2];
    double hx = plan->mesh_h[0], hy = plan->mesh_h[1], hz = plan->mesh_h[2];
    const int64_t n3 = int64_t(g.n) * g.n * g.n;
    hipError_t e = hipSuccess;
    for (;;) {
        MgLevel L;
        L.G.ncells = int64_t(mx) * my * mz;
        L.G.offset = 0;
        L.G.logB = g.logB;
        L.G.mx = mx;
        L.G.my = my;
        L.G.mz = mz;
        L.G.sx = hy * hz / hx;
        L.G.sy = hx * hz / hy;
        L.G.sz = hx * hy / hz;
        const int64_t B = int64_t(1) << g.logB;
        L.elems = (L.G.ncells + B - 1) / B * n3 * B;
        const size_t vb = static_cast<size_t>(L.elems) * es;
        if (e == hipSuccess) e = hipMalloc(&L.t, vb);
        // the finest level works on the caller's b and u, except with FP32
        // storage, whose finest level has its own FP32 copies
        if (!m->lv.empty() || storage == TP_F32) {
            if (e == hipSuccess) e = hipMalloc(&L.b, vb);
            if (e == hipSuccess) e = hipMalloc(&L.u, vb);
        }
        m->lv.push_back(L);
        if (e != hipSuccess || mx % 2 || my % 2 || mz % 2) break;
        mx /= 2, my /= 2, mz /= 2;
        hx *= 2, hy *= 2, hz *= 2;
    }
    if (e != hipSuccess) {
        free_mg(m);
        delete m;
        (void)hipGetLastError();
        return set_error(TP_ERR_OOM, "multigrid workspace allocation failed");
    }
    const MgLevel& Lc = m->lv.back();
    m->n0 = Lc.G.ncells * n3;
    if (m->n0 > kMaxCoarse && g.n > kLaneMaxN && Lc.G.ncells * 8 <= kMaxCoarse) {
        // too large for the dense solve at degree p: one more level of
        // degree 1 on the same cells (Lagrange basis; n >= 5 only)
        m->deg = true;
        m->n0 = Lc.G.ncells * 8;
        const size_t cb = static_cast<size_t>(m->n0) * sizeof(double);
        e = hipMalloc(reinterpret_cast<void**>(&m->deg_b), cb);
        if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&m->deg_u), cb);
        if (e != hipSuccess) {
            free_mg(m);
            delete m;
            (void)hipGetLastError();
            return set_error(TP_ERR_OOM, "multigrid workspace allocation failed");
        }
    }
    if (m->n0 > kMaxCoarse) {
        free_mg(m);
        delete m;
        return set_error(TP_ERR_UNSUPPORTED, "the coarsest level (" + std::to_string(m->n0) +
                                                 " unknowns) is too large for its dense solve");
    }
    if (m->lv.size() == 1 && !m->lv[0].b && !m->deg) {   // no coarser level: the finest is solved densely; it needs b and u scratch
        MgLevel& L0 = m->lv[0];
        const size_t vb = static_cast<size_t>(L0.elems) * es;
        e = hipMalloc(&L0.b, vb);
        if (e == hipSuccess) e = hipMalloc(&L0.u, vb);
        if (e != hipSuccess) {
            free_mg(m);
            delete m;
            (void)hipGetLastError();
            return set_error(TP_ERR_OOM, "multigrid workspace allocation failed");
        }
    }
    // the coarse inverse, shared per device and coarsest level
    int dev = 0;
    (void)hipGetDevice(&dev);
    const CoarseKey key{dev, g.n, plan->basis, m->deg ? 1 : 0, Lc.G.mx, Lc.G.my, Lc.G.mz, hx, hy, hz, plan->penalty_C};
    std::lock_guard<std::mutex> lock(g_coarse_mutex);
    auto it = g_coarse.find(key);
    if (it != g_coarse.end()) {
        m->coarse_inv = it->second;
    } else {
        std::vector<double> A, inv;
        tp_status st = TP_OK;
        if (m->deg) {
            switch (g.n) {
                case 5: st = coarse_probe_deg<5>(m, A); break;
                case 6: st = coarse_probe_deg<6>(m, A); break;
                case 7: st = coarse_probe_deg<7>(m, A); break;
                default: st = coarse_probe_deg<8>(m, A); break;
            }
        } else {
            switch (g.n) {
                case 2: st = coarse_probe_n<2>(m, A); break;
                case 3: st = coarse_probe_n<3>(m, A); break;
                case 4: st = coarse_probe_n<4>(m, A); break;
                case 5: st = coarse_probe_n<5>(m, A); break;
                case 6: st = coarse_probe_n<6>(m, A); break;
                case 7: st = coarse_probe_n<7>(m, A); break;
                default: st = coarse_probe_n<8>(m, A); break;
            }
        }
        if (st == TP_OK && !spd_inverse(m->n0, A, inv))
            st = set_error(TP_ERR_NOT_SPD, "the coarsest level operator is not positive definite");
        double* dinv = nullptr;
        if (st == TP_OK) {
            e = hipMalloc(reinterpret_cast<void**>(&dinv), inv.size() * sizeof(double));
            if (e == hipSuccess)
                e = hipMemcpy(dinv, inv.data(), inv.size() * sizeof(double), hipMemcpyHostToDevice);
            if (e != hipSuccess) st = hip_error(e, "coarse inverse upload");
        }
        if (st != TP_OK) {
            if (dinv) (void)hipFree(dinv);
            free_mg(m);
            delete m;
            return st;
        }
        g_coarse[key] = dinv;
        m->coarse_inv = dinv;
    }
    *out = m;
    return TP_OK;
}

tp_status tp_mg_vcycle(tp_mg* m, const double* b, double* x, hipStream_t stream) {
    if (!m) return set_error(TP_ERR_ARG, "multigrid is null");
    if (!b || !x) return set_error(TP_ERR_ARG, "b and x must be non-null");
    if (static_cast<const void*>(b) == static_cast<const void*>(x)) return set_error(TP_ERR_ARG, "b and x must not alias");
    return mg_enqueue_vcycle(m, b, x, false, stream);
}

tp_status tp_mg_destroy(tp_mg* m) {
    if (!m) return TP_OK;
    free_mg(m);
    delete m;
    return TP_OK;
}

}  // extern "C"
