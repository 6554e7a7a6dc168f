// Element and quadrature-point helpers shared by the assembly kernels
// (internal header of libvms, gfx950).
#pragma once
#include "geom.h"
#include "kernels.h"

namespace vmsk {
using namespace vmsd;

__device__ inline const double *field_in(const AsmArgs &a, int f) {
    switch (f) {
        case 0: return a.f[0];
        case 1: return a.f[1];
        case 2: return a.f[2];
        case 3: return a.f[3];
        case 4: return a.f[4];
        case 5: return a.f[5];
        default: return a.f[6];
    }
}

// reference coordinates (double) and weight of point pt of the item
template <bool SUB>
__device__ inline void point_xw(const AsmArgs &a, uint32_t en, int pt, double h, double xi[3],
                                double &w) {
    if (!SUB) {
        for (int k = 0; k < 3; ++k) xi[k] = ((pt >> k) & 1) ? VMS_XI : -VMS_XI;
        const double hh = 0.5 * h;
        w = hh * hh * hh;
        return;
    }
    const int l = (int)(en & 3u), D = a.depth;
    const uint32_t key = en >> 2;
    const int gp = (int)((key >> (3 * (D - l))) & 7u);
    const double sl = ldexp(1.0, -l);
    for (int ax = 0; ax < 3; ++ax) {
        double f = 0.0;
        for (int k = 1; k <= l; ++k)
            if ((key >> (3 * (D - k + 1) + ax)) & 1u) f += ldexp(1.0, -k);
        f = __dadd_rn(f, sl * (((gp >> ax) & 1) ? VMS_GP : VMS_GM));
        xi[ax] = __dsub_rn(2.0 * f, 1.0);
    }
    const double hs = h * ldexp(1.0, -(l + 1));
    w = hs * hs * hs;
}

}  // namespace vmsk
