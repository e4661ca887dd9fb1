// The pixel decision of the far-field ray kernel: plain arithmetic, shared with its CPU tests.
#pragma once

#include <cmath>
#include <cstdint>

#include "rs_layout.h"

namespace rs {

// The pixel of an npx x npy map (fewer than 2^31 pixels) that the position (u, v), in pixels, is
// inside by more than the bounds Mu, Mv on its error, or -1. A position outside the map, or one
// that is not finite, is not converted to a whole number: -1.
RS_HOST_DEVICE inline int pixel_inside(double u, double v, double Mu, double Mv, int64_t npx, int64_t npy) {
    const double fu = floor(u), fv = floor(v);
    const double ru = u - fu, rv = v - fv;   // exact
    const bool in = fu >= 0.0 && fu < (double)npx && fv >= 0.0 && fv < (double)npy && ru > Mu && ru + Mu < 1.0 &&
                    rv > Mv && rv + Mv < 1.0;
    return in ? (int)((uint32_t)(int)fv * (uint32_t)npx + (uint32_t)(int)fu) : -1;
}

}  // namespace rs
