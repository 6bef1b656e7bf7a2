// Kernel instantiations for the D3Q19 lattice.
#define LBM_Q 19
#include "lbm_dispatch.h"

namespace lbm {

hipError_t launch_sweep_q19(const Dims &dm, const Geom &g, const void *coefs, const void *fin,
                            void *fout, const void *pin, void *pout, int *flag, hipStream_t st) {
    LBM_BY_PREC(sweep_typed, dm, g, coefs, fin, fout, pin, pout, flag, st)
}

hipError_t launch_init_q19(const Dims &dm, const Geom &g, const void *coefs, const double *phi0,
                           void *f, void *p, const double *rfield, hipStream_t st) {
    LBM_BY_PREC(init_typed, dm, g, coefs, phi0, f, p, rfield, st)
}

hipError_t launch_phi_q19(const Dims &dm, const Geom &g, const void *coefs, const void *f,
                          double *phi, const double *rfield, hipStream_t st) {
    LBM_BY_PREC(phi_typed, dm, g, coefs, f, phi, rfield, st)
}

hipError_t launch_phi_reduce_q19(const Dims &dm, const Geom &g, const void *coefs, const void *f, const double *ref,
                               const double *rfield, double *part, int nparts, double *out, hipStream_t st) {
    LBM_BY_PREC(phi_reduce_typed, dm, g, coefs, f, ref, rfield, part, nparts, out, st)
}

hipError_t launch_sweep_gen_q19(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout,
                               const void *pin, void *pout, int *flag, const double *kfield, const double *rfield,
                               bool remark3, hipStream_t st) {
    LBM_BY_PREC(sweep_gen_typed, dm, g, coefs, fin, fout, pin, pout, flag, kfield, rfield, remark3, st)
}

hipError_t launch_recenter_q19(const Dims &dm, const Geom &g, void *coefs, void *f, void *p, double *part,
                              int nparts, double *shift, hipStream_t st) {
    LBM_BY_PREC(recenter_typed, dm, g, coefs, f, p, part, nparts, shift, st)
}


hipError_t launch_adjoint_q19(const Dims &dm, const Geom &g, const void *coefs, const void *f, const void *p,
                              const void *psi_next, const double *pi_next, void *psi_out, double *pi_out,
                              double *gk_part, hipStream_t st) {
    LBM_BY_PREC_ADJ(adjoint_typed, dm, g, coefs, f, p, psi_next, pi_next, psi_out, pi_out, gk_part, st)
}

hipError_t launch_adjoint_init_q19(const Dims &dm, const Geom &g, const void *coefs, const double *phi0,
                                   const void *psi0, const double *pi0, double *out, hipStream_t st) {
    LBM_BY_PREC_ADJ(adjoint_init_typed, dm, g, coefs, phi0, psi0, pi0, out, st)
}

hipError_t launch_seed_q19(const Dims &dm, const Geom &g, const double *gphi, void *psi, double *pi,
                           hipStream_t st) {
    LBM_BY_PREC_ADJ(seed_typed, dm, g, gphi, psi, pi, st)
}


hipError_t launch_set_wall_q19(const Dims &dm, void *coefs, const double *ewp, hipStream_t st) {
    LBM_BY_PREC(set_wall_typed, dm, coefs, ewp, st)
}

hipError_t launch_sweep2_q19(const Dims &dm, const Geom &g, const void *coefs, const void *fin, void *fout,
                             const void *pin, void *pout, int *flag, int shape, uint32_t zc, hipStream_t st) {
    LBM_BY_PREC(sweep2_3d_typed, dm, g, coefs, fin, fout, pin, pout, flag, shape, zc, st, nullptr)
}

hipError_t sweep2_q19_occupancy(const Dims &dm, const Geom &g, int shape, int *blocks_per_cu) {
    LBM_BY_PREC(sweep2_3d_typed, dm, g, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, shape, 1u, nullptr,
                blocks_per_cu)
}

bool two_step3_shape_of(int prec, int shape, int *rows, int *waves) {
    int r = 0, w = 0;
    const bool ok = prec == 0 ? two_step3_shape<double>(shape, r, w) : two_step3_shape<float>(shape, r, w);
    if (ok) { *rows = r; *waves = w; }
    return ok;
}

}  // namespace lbm
