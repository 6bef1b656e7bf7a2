// D2Q9 passes of several time steps, FP64 storage.
#include "lbm_multi_dispatch.h"

namespace lbm {

hipError_t launch_sweep_multi_q9_f64(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout,
                                     const void *pin, void *pout, int *flag, int shape, hipStream_t st) {
    return multi_typed<double, double, 32, 16, 8>(dm, g, coefs, fin, fout, pin, pout, flag, shape, st);
}

hipError_t launch_sweep_multi_q9(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout,
                                 const void *pin, void *pout, int *flag, int shape, hipStream_t st) {
    if (!dm.deg3 || !dm.o32) return hipErrorNotSupported;
    // a Scheme-A source reads the history pin and writes pout (distinct)
    if (dm.src && !dm.sb && (!pin || !pout || pin == pout)) return hipErrorInvalidValue;
    switch (dm.prec) {
        case 0: return launch_sweep_multi_q9_f64(dm, g, coefs, fin, fout, pin, pout, flag, shape, st);
        case 1: return launch_sweep_multi_q9_f32(dm, g, coefs, fin, fout, pin, pout, flag, shape, st);
        case 2: return launch_sweep_multi_q9_f16(dm, g, coefs, fin, fout, pin, pout, flag, shape, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
