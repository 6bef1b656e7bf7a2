// Template dispatch of the D2Q9 passes of several time steps; included by one
// translation unit per storage type (sweep_multi_q9_*.hip).
#pragma once

#include "lbm_multi.h"

namespace lbm {

template <typename TS, typename TC, int T, int TR, int NW, int TX = 64>
hipError_t multi_shape(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout, const void *pin,
                       void *pout, int *flag, hipStream_t st) {
    using TP = typename HistType<TS>::T;
    constexpr uint32_t TW = TX - 2 * (T - 1), TH = TR - 2 * (T - 1);
    const uint32_t tiles_x = (g.nx + TW - 1) / TW, tiles_y = (g.ny + TH - 1) / TH;
    const dim3 grid(tiles_x * tiles_y), block(64 * NW);
    // source: none, Scheme A (history pin -> pout) or Scheme B (no history)
    // collision: moment space, equal rates, rates 1.  The last saves 9 of 106
    // operations of a node where issue is the bound (us per step with a source:
    // FP32 1024^2 6.20 -> 5.84, 4000 x 2500 50.1 -> 46.2; FP64 1024^2 12.28 ->
    // 11.95; FP16 4000 x 2500 44.7 -> 41.6)
    const int code = (dm.sb ? 2 : (dm.src ? 1 : 0)) * 12 + (dm.kvar ? 6 : 0) + (dm.wall ? 3 : 0) +
                     (dm.unit ? 2 : (dm.eqr ? 1 : 0));
#define LBM_MULTI(S, K, W, E)                                                                             \
    case (S * 12 + K * 6 + W * 3 + E):                                                                    \
        hipLaunchKernelGGL((k_sweep_multi<TS, TC, S == 1, K, T, TR, NW, S == 2, W, E, TX>), grid, block, 0, st, g, \
                           (const Coefs<TC> *)coefs, (const TS *)fin, (TS *)fout, (const TP *)pin, (TP *)pout, \
                           tiles_x, flag);                                                                \
        break;
#define LBM_MULTI4(S, K) LBM_MULTI(S, K, 0, 1) LBM_MULTI(S, K, 0, 2) LBM_MULTI(S, K, 1, 1) LBM_MULTI(S, K, 1, 2)
#define LBM_MULTI6(S, K) LBM_MULTI(S, K, 0, 0) LBM_MULTI(S, K, 1, 0) LBM_MULTI4(S, K)
    switch (code) {
        LBM_MULTI6(0, 0) LBM_MULTI6(0, 1) LBM_MULTI6(1, 0) LBM_MULTI6(1, 1)
        // Scheme B with unequal rates runs the general sweep (general_path)
        LBM_MULTI4(2, 0) LBM_MULTI4(2, 1)
        default: return hipErrorInvalidValue;
    }
#undef LBM_MULTI6
#undef LBM_MULTI4
#undef LBM_MULTI
    return hipGetLastError();
}

// The shapes of multi_shape_of: shape 3 runs on R3 rows, shape 4 on R4
// rows with N4 waves.
template <typename TS, typename TC, int R3, int R4, int N4>
hipError_t multi_typed(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout, const void *pin,
                       void *pout, int *flag, int shape, hipStream_t st) {
    switch (shape) {
        case 0: return multi_shape<TS, TC, 8, 16, 16>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        case 1: return multi_shape<TS, TC, 6, 16, 16>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        case 2: return multi_shape<TS, TC, 4, 16, 16>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        case 3: return multi_shape<TS, TC, 6, R3, 16>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        case 4: return multi_shape<TS, TC, 4, R4, N4>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        case 5: return multi_shape<TS, TC, 8, 16, 8, 32>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        case 6: return multi_shape<TS, TC, 6, 16, 8, 32>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        case 7: return multi_shape<TS, TC, 4, 16, 8, 32>(dm, g, coefs, fin, fout, pin, pout, flag, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
