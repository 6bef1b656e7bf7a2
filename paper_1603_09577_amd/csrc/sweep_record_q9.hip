// D2Q9 passes of several time steps that record every state.
#include "lbm_multi.h"

namespace lbm {

namespace {

template <typename TS, typename TC, int T, int TR, int NW>
hipError_t record_shape(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout, size_t f_step,
                        const void *pin, void *pout, size_t p_step, int *flag, hipStream_t st) {
    using TP = typename HistType<TS>::T;
    constexpr uint32_t TW = 64 - 2 * (T - 1), TH = TR - 2 * (T - 1);
    const uint32_t tiles_x = (g.nx + TW - 1) / TW, tiles_y = (g.ny + TH - 1) / TH;
    const dim3 grid(tiles_x * tiles_y), block(64 * NW);
    const int code = (dm.unit ? 8 : 0) + (dm.src ? 4 : 0) + (dm.kvar ? 2 : 0) + (dm.wall ? 1 : 0);
#define LBM_RECE(S, K, W, E)                                                                                \
    case ((E == 2 ? 8 : 0) + S * 4 + K * 2 + W):                                                                           \
        hipLaunchKernelGGL((k_sweep_record<TS, TC, S, K, T, TR, NW, W, E>), grid, block, 0, st, g,           \
                           (const Coefs<TC> *)coefs, (const TS *)fin, (TS *)fout, (uint64_t)(f_step / sizeof(TS)), \
                           (const TP *)pin, (TP *)pout, (uint64_t)(p_step / sizeof(TP)), tiles_x, flag);  \
        break;
#define LBM_REC(S, K, W) LBM_RECE(S, K, W, 1) LBM_RECE(S, K, W, 2)
    switch (code) {
        LBM_REC(0, 0, 0) LBM_REC(0, 0, 1) LBM_REC(0, 1, 0) LBM_REC(0, 1, 1)
        LBM_REC(1, 0, 0) LBM_REC(1, 0, 1) LBM_REC(1, 1, 0) LBM_REC(1, 1, 1)
        default: return hipErrorInvalidValue;
    }
#undef LBM_REC
#undef LBM_RECE
    return hipGetLastError();
}

}  // namespace

hipError_t launch_sweep_record_q9(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout,
                                  size_t f_step, const void *pin, void *pout, size_t p_step, int *flag, int steps,
                                  bool tall, hipStream_t st) {
    if (!dm.deg3 || !dm.o32 || !dm.eqr || dm.sb || dm.prec > 1) return hipErrorNotSupported;
    if (dm.src && (!pin || !pout || pin == pout)) return hipErrorInvalidValue;
#define LBM_RECS(TS, TC, T, TR, NW) \
    return record_shape<TS, TC, T, TR, NW>(dm, g, coefs, fin, fout, f_step, pin, pout, p_step, flag, st)
    if (dm.prec == 0) {
        if (steps == 6) { if (tall) LBM_RECS(double, double, 6, 32, 16); LBM_RECS(double, double, 6, 16, 16); }
        if (steps == 4) { if (tall) LBM_RECS(double, double, 4, 16, 8); LBM_RECS(double, double, 4, 16, 16); }
    } else {
        if (steps == 6) { if (tall) LBM_RECS(float, float, 6, 32, 16); LBM_RECS(float, float, 6, 16, 16); }
        if (steps == 4) { if (tall) LBM_RECS(float, float, 4, 32, 16); LBM_RECS(float, float, 4, 16, 16); }
    }
#undef LBM_RECS
    return hipErrorInvalidValue;
}

}  // namespace lbm
