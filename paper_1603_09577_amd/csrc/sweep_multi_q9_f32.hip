// D2Q9 passes of several time steps, FP32 storage.
#include "lbm_multi_dispatch.h"

namespace lbm {

hipError_t launch_sweep_multi_q9_f32(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout,
                                     const void *pin, void *pout, int *flag, int shape, hipStream_t st) {
    return multi_typed<float, float, 32, 32, 16>(dm, g, coefs, fin, fout, pin, pout, flag, shape, st);
}

}  // namespace lbm
