// Constants and geometry shared by the cosmic-shear forward and
// adjoint kernels (App. A of the paper).
#pragma once

#include "devutil.h"
#include "nsmi.h"

namespace nsmi {

constexpr double C_KM_S = 299792.458;                 // speed of light [km/s]
constexpr double C1_RHOCR = 5e-14 * 2.77536627e11;    // C1 rho_cr of the NLA model (Eq. A4)
constexpr double GROWTH_INDEX = 0.55;
constexpr double LN10 = 2.302585092994045684;
constexpr int MAXB = 10;                              // tomographic bins supported by the kernels

struct ShearGeom {
    int n_a, n_z, n_k, n_ell, n_bins, n_pairs;
    double a_min, da, zmax, k_min, k_max, u0, du, nz_sigma;
    double u1;        // log10 k_max
};

ShearGeom shear_geom(const ns_model* m);

}  // namespace nsmi
