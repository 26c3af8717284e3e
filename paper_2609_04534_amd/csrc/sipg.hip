// Launch of the coupled SIPG operator of a mesh plan (device code in sipg.h).
#include "sipg.h"

namespace tpfdm {

namespace {

// 64 W cells per workgroup of N waves (n <= 4).  u is read with cached
// loads (a block is also a face source of its neighbours); v is streamed out.
template <int N, typename TS, typename TC, int W, bool NT, int LB, bool HERM = false>
__global__ __launch_bounds__(64 * N, (tile_waves<N, TC, W>())) void k_sipg_tile(const TS* __restrict__ u,
                                                                                TS* __restrict__ v, MeshArgs G,
                                                                                TileTab<N, TC, HERM> R) {
    constexpr int N2 = N * N, N3 = N * N * N;
    __shared__ Cells<TC, W> A[N3][64];
    const TileCell<W> T(G, lane_tile(blockIdx.x, gridDim.x, plane_tiles<N, TS, W>(G)));
    Cells<TC, W> out[N2];
    tile_sipg<N, TS, TC, W, LB, HERM>(u, G, R, T, A, out);
    if (!T.valid) return;
    const int lb = LB >= 0 ? LB : G.logB;
    TS* vb = v + G.offset + block_base(T.c, lb, N3) + (static_cast<int64_t>(T.w * N2) << lb);
#pragma unroll
    for (int q = 0; q < N2; ++q) st_cells<NT>(vb + (static_cast<int64_t>(q) << lb), out[q]);
}

// Waves per workgroup of the one-cell-per-wave kernel.  From B = 8 on the cells
// of a layout tile share every cache line of their blocks, so eight neighbours
// run on one CU and its vector cache serves a line to all of them; one to a
// workgroup, each CU fetched the line for one cell.  28^3 cells, FP64, one wave
// against eight: B = 8 n = 6 86 / 70 us, n = 8 302 / 170 us; B = 64 n = 6 134 /
// 92 us, n = 8 480 / 303 us.  Below kTileCells cells too few CUs get any (B = 8,
// FP64, n = 8: 512 cells 11 / 16 us, 1452 cells 24 / 18 us).
constexpr int kTileWaves = 8;
constexpr int64_t kTileCells = 1024;

// One cell per wave (n >= 5); HERM: the Hermite-type basis.
template <int N, typename T, bool VP, bool HERM, int WV = 1>
__global__ __launch_bounds__(64 * WV, 2) void k_sipg_wave(const T* __restrict__ u, T* __restrict__ v, MeshArgs G,
                                                  const T* __restrict__ tab, WaveFace<N, T> F) {
    constexpr int TAB = 2 * (EOShape<N>::SE + EOShape<N>::SO);
    __shared__ WaveLds<N, T> L[WV];
    const int wave = WV == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.y);
    // FP64: the tables are read at wave-uniform global addresses (scalar
    // loads; in VGPRs they would take half the register file, from LDS they
    // would compete with the slab traffic); FP32: from registers
    T TB[sizeof(T) == 8 ? 1 : TAB];
    const T* tb = TB;
    if constexpr (sizeof(T) == 8) {
        tb = tab;
    } else {
        load_table<T, TAB>(TB, tab, nullptr);   // FP32: straight from the global table
    }
    const int64_t c = static_cast<int64_t>(wave_tile<WV>(blockIdx.x, gridDim.x, G)) * WV + wave;
    if (WV > 1 && c >= G.ncells) return;   // (waves of a workgroup share nothing)
    T y[N];
    wave_sipg_cell<N, T, VP, HERM>(u, G, tb, F, c, L[wave], y);
    const Pencil<N> pc(1);
    if (pc.act) {
        T* vb = v + G.offset + block_base(c, G.logB, N * N * N);
        // streamed where a plane is whole lines of this cell alone
        constexpr bool kWholeLines = WV == 1 && (N * N * sizeof(T)) % 128 == 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            T* o = vb + (static_cast<int64_t>((i * N + pc.pa) * N + pc.pb) << G.logB);
            if constexpr (kWholeLines) stg(o, y[i]);
            else stc(o, y[i]);
        }
    }
}

tp_status check_launch(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, what);
    return TP_OK;
}
template <int N, typename TS, typename TC, bool HERM>
tp_status sipg_tile_n(const Plan& plan, const MeshArgs& G, bool face_only, const void* u, void* v, hipStream_t s) {
    const TileTab<N, TC, HERM> R = tile_tab<N, TC, HERM>(plan, face_only);
    const TS* ui = static_cast<const TS*>(u);
    TS* vo = static_cast<TS*>(v);
    const bool aligned = reinterpret_cast<uintptr_t>(u) % 16 == 0 && reinterpret_cast<uintptr_t>(v) % 16 == 0;
    const dim3 wg(64, N);
    if (tile_pairs(G, sizeof(TS), aligned)) {
        if constexpr (sizeof(TS) == 8)
            hipLaunchKernelGGL((k_sipg_tile<N, TS, TC, 2, true, 6, HERM>), dim3(tile_grid(G, 2)), wg, 0, s, ui, vo, G,
                               R);
    } else if (G.logB == 6) {
        hipLaunchKernelGGL((k_sipg_tile<N, TS, TC, 1, true, 6, HERM>), dim3(tile_grid(G, 1)), wg, 0, s, ui, vo, G, R);
    } else if (lane_whole_lines<TS>(G.logB)) {
        hipLaunchKernelGGL((k_sipg_tile<N, TS, TC, 1, true, -1, HERM>), dim3(tile_grid(G, 1)), wg, 0, s, ui, vo, G, R);
    } else {
        hipLaunchKernelGGL((k_sipg_tile<N, TS, TC, 1, false, -1, HERM>), dim3(tile_grid(G, 1)), wg, 0, s, ui, vo, G,
                           R);
    }
    return check_launch("SIPG apply launch");
}

template <int N, typename T>
tp_status sipg_wave_n(const Plan& plan, const MeshArgs& G, bool face_only, const void* u, void* v, hipStream_t s) {
    const WaveFace<N, T> F = wave_face<N, T>(plan);
    const T* tab = reinterpret_cast<const T*>(eo_table(plan, N, face_only ? EO_APPLY_F : EO_APPLY_A,
                                                       sizeof(T) == 8 ? 0 : 1));
    const unsigned grid = static_cast<unsigned>(G.ncells);
    const T* ui = static_cast<const T*>(u);
    T* vo = static_cast<T*>(v);
    // 16-byte pencils: block-contiguous layout and an aligned vector
    const bool vp = G.logB == 0 && (reinterpret_cast<uintptr_t>(ui + G.offset) % 16 == 0) &&
                    (N * sizeof(T)) % 16 == 0;
    auto launch = [&](auto Hc) {
        constexpr bool HERM = decltype(Hc)::value;
        if (vp)
            hipLaunchKernelGGL((k_sipg_wave<N, T, true, HERM>), dim3(grid), dim3(64), 0, s, ui, vo, G, tab, F);
        else if (G.logB < 3 || G.ncells < kTileCells)
            hipLaunchKernelGGL((k_sipg_wave<N, T, false, HERM>), dim3(grid), dim3(64), 0, s, ui, vo, G, tab, F);
        else
            hipLaunchKernelGGL((k_sipg_wave<N, T, false, HERM, kTileWaves>), dim3((grid + kTileWaves - 1) / kTileWaves),
                               dim3(64, kTileWaves), 0, s, ui, vo, G, tab, F);
    };
    if (plan.basis == TP_BASIS_HERMITE) launch(std::true_type{});
    else launch(std::false_type{});
    return check_launch("SIPG apply launch");
}

template <typename TS, typename TC>
tp_status sipg_dispatch(const Plan& plan, const MeshArgs& G, int n, bool face_only, const void* u, void* v,
                        hipStream_t s) {
    switch (n) {
        case 2: return sipg_tile_n<2, TS, TC, false>(plan, G, face_only, u, v, s);
        case 3: return sipg_tile_n<3, TS, TC, false>(plan, G, face_only, u, v, s);
        case 4:   // the Hermite-type basis has n >= 4: two-layer face terms
            return plan.basis == TP_BASIS_HERMITE ? sipg_tile_n<4, TS, TC, true>(plan, G, face_only, u, v, s)
                                                  : sipg_tile_n<4, TS, TC, false>(plan, G, face_only, u, v, s);
        case 5: return sipg_wave_n<5, TC>(plan, G, face_only, u, v, s);
        case 6: return sipg_wave_n<6, TC>(plan, G, face_only, u, v, s);
        case 7: return sipg_wave_n<7, TC>(plan, G, face_only, u, v, s);
        case 8: return sipg_wave_n<8, TC>(plan, G, face_only, u, v, s);
        default: break;
    }
    return set_error(TP_ERR_UNSUPPORTED, "unsupported n");
}

}  // namespace

tp_status launch_sipg(const Plan& plan, const GroupInfo& g, bool face_only, const void* u, void* v, tp_dtype dt,
                      hipStream_t s) {
    if (g.nblocks == 0) return TP_OK;
    const MeshArgs G = mesh_args(plan, g);
    switch (dt) {
        case TP_F64: return sipg_dispatch<double, double>(plan, G, g.n, face_only, u, v, s);
        case TP_F32: return sipg_dispatch<float, float>(plan, G, g.n, face_only, u, v, s);
        default: break;
    }
    return set_error(TP_ERR_UNSUPPORTED, "the SIPG operator supports TP_F64 and TP_F32");
}

}  // namespace tpfdm
