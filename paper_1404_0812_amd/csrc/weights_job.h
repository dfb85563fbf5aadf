// Plain-data description of one weights job (host and device).
#pragma once

#include <cstdint>

#define RBW_RMAX 10

namespace rbw {

struct WOpts {
    int n, kernel, degree, mode;
    double eps_fixed, kappa_target, eps_tol, br_lo, br_hi, band_lo, band_hi, rank_tol;
    int band_stop, max_expand;
    double band_rel;  // multisection precision of a kappa found inside the band
};

// One stencil set: inputs, options and outputs (device pointers).
struct Job {
    WOpts o;
    int64_t N;
    const double* xyz;
    const double* nrm;
    const int32_t* idx;
    const double* eps_in;
    double* w;
    double* eps;
    double* kappa;
    int32_t* status;
    int32_t* nevals;
    int kappa_only;
};

#ifdef __HIPCC__
__host__ __device__
#endif
inline int border_cols(int degree) { return degree == 0 ? 1 : (degree == 1 ? 4 : 10); }

// Tiling of the weights kernels: the smallest that holds n + border rows.
inline int tiling(const WOpts& o) {
    const int m = o.n + border_cols(o.degree);
    return m <= 32 ? 32 : (m <= 48 ? 48 : (m <= 64 ? 64 : 128));
}
// The persistent launches have no half-wavefront form: m <= 32 runs there as
// m <= 48.  The halves leave a loop over an item's stencils at different turns,
// so its counter is a vector register, live across the whole of
// process_stencil, and spilled; the compiler reloaded it where branches meet,
// ahead of the instruction that restores the mask of active lanes.  With no
// lane active there nothing was reloaded, and the loop went on from whatever
// the register held, to stencils that do not exist (a GPU fault).
inline int batch_tiling(const WOpts& o) { return tiling(o) < 48 ? 48 : tiling(o); }

}  // namespace rbw
