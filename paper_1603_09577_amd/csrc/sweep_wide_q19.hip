// D3Q19 passes of two time steps in columns of 64-node lines.
#include "lbm_wide3.h"

namespace lbm {

namespace {

// occ != nullptr: launch nothing and report the kernel's resident workgroups
// per CU instead (the z-chunk choice needs it).
template <typename TS, typename TC, int TY>
hipError_t wide_typed(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout, const void *pin,
                      void *pout, int *flag, uint32_t zc, hipStream_t st, int *occ) {
    using TP = typename HistType<TS>::T;
    const uint32_t tiles_x = (g.nx + 63) / 64, tiles_y = (g.ny + TY - 1) / TY, tiles_z = (g.nz + zc - 1) / zc;
    const dim3 grid(tiles_x * tiles_y * tiles_z), block(64 * (TY + 3));
    // source: none, Scheme B (no history) or Scheme A (history pin -> pout)
    // kernels for rates 1 apart: us per step 128^3 FP64 with a source 96.7 -> 91.3,
    // FP16 33 -> 31; 256^3 FP32, bound by memory, 269 -> 267
    const int code = (dm.unit ? 12 : 0) + (dm.sb ? 1 : (dm.src ? 2 : 0)) * 4 + (dm.kvar ? 2 : 0) + (dm.wall ? 1 : 0);
#define LBM_W3E(S, K, W, E)                                                                                   \
    case ((E == 2 ? 12 : 0) + S * 4 + K * 2 + W):                                                         \
        if (occ)                                                                                          \
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(                                          \
                occ, k_sweep2_3dw<TS, TC, K, W, 3, TY, S == 1, S == 2, E>, 64 * (TY + 3), 0);          \
        hipLaunchKernelGGL((k_sweep2_3dw<TS, TC, K, W, 3, TY, S == 1, S == 2, E>), grid, block, 0, st, g, \
                           (const Coefs<TC> *)coefs, (const TS *)fin, (TS *)fout, (const TP *)pin, (TP *)pout, \
                           tiles_x, tiles_y, zc, flag);                                                   \
        break;
#define LBM_W3(S, K, W) LBM_W3E(S, K, W, 1) LBM_W3E(S, K, W, 2)
    switch (code) {
        LBM_W3(0, 0, 0) LBM_W3(0, 0, 1) LBM_W3(0, 1, 0) LBM_W3(0, 1, 1)
        LBM_W3(1, 0, 0) LBM_W3(1, 0, 1) LBM_W3(1, 1, 0) LBM_W3(1, 1, 1)
        LBM_W3(2, 0, 0) LBM_W3(2, 0, 1) LBM_W3(2, 1, 0) LBM_W3(2, 1, 1)
        default: return hipErrorInvalidValue;
    }
#undef LBM_W3
#undef LBM_W3E
    return hipGetLastError();
}

hipError_t wide_any(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout, const void *pin,
                    void *pout, int *flag, uint32_t zc, hipStream_t st, int *occ) {
    if (!dm.deg3 || !dm.o32 || !dm.eqr || zc < 1) return hipErrorNotSupported;
    // a Scheme-A source reads the history pin and writes pout (distinct)
    if (!occ && dm.src && !dm.sb && (!pin || !pout || pin == pout)) return hipErrorInvalidValue;
    switch (dm.prec) {
        case 0: return wide_typed<double, double, 6>(dm, g, coefs, fin, fout, pin, pout, flag, zc, st, occ);
        case 1: return wide_typed<float, float, 13>(dm, g, coefs, fin, fout, pin, pout, flag, zc, st, occ);
        case 2: return wide_typed<_Float16, float, 13>(dm, g, coefs, fin, fout, pin, pout, flag, zc, st, occ);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_sweep2w_q19(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout,
                              const void *pin, void *pout, int *flag, uint32_t zc, hipStream_t st) {
    return wide_any(dm, g, coefs, fin, fout, pin, pout, flag, zc, st, nullptr);
}

hipError_t sweep2w_q19_occupancy(const Dims &dm, const Geom &g, int *blocks_per_cu) {
    return wide_any(dm, g, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 1u, nullptr, blocks_per_cu);
}

}  // namespace lbm
